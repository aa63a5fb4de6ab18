// Training-step kernels of improved targeted dropout (Sec. 5.1; schedule of
// Sec. 6) for a CCI layer.
//
// cci_td_mask: candidate dropout of one step.  One lane per (group g,
// column c), as in the projection: the lane ranks the G weights of its group
// by magnitude (larger |w| first, ties to the lower row), marks the n_target
// lowest as candidates, and drops a candidate when the caller's random word
// for it is below floor(drop_rate * 2^32).  HBM-bound: reads W and the random
// words, writes W_eff and the keep mask, all coalesced along c.  Ranking 16
// rows against each other took 480 vector instructions a lane; the n_target-th
// smallest magnitude now comes from a sorting network (63 compare-exchanges for
// 16 rows).  The streamed operands displace each other in the caches, so rows
// that start on whole 128-byte lines are read non-temporally (a line shared
// by two rows would be fetched twice), unless nothing is a candidate: then the
// random words are not read and W alone stays resident between calls.  us, all
// pairs compared / sorted / sorted and non-temporal, operands from memory and
// (in brackets) left in the caches by the call before: 4096 x 4096, G = 16
// 46.0 / 38.7 / 33.9 (36.8 / 32.2 / 33.0); G = 2 47.7 / 38.9 / 35.5 (33.8 /
// 31.6 / 33.6); 3072 x 3333, G = 8 33.0 / 29.2 / 27.1 (24.9 / 24.1 / 27.9).
//
// cci_grad_packed: gradient of the packed values once the mask is fixed,
//   dvals[g][k][c] = sum_n dY[n][gG + idx[g][k][c]] * X[n][c].
// (bf16 operands in the shapes it takes run on the matrix cores instead:
// cci_grad.hip.  This kernel serves fp32, short reductions and other shapes.)
// A workgroup owns four consecutive groups and 256 columns (a lane per
// column, its indices in registers); per pass of up to 32 rows the rows of dY
// restricted to those groups' outputs and of X restricted to the columns are
// staged in LDS with every load in flight, then each lane gathers the
// entries its indices name (one LDS read and one FMA per kept weight and row).
// Only kept weights are touched: N * nnz multiply-adds on the vector ALUs.
#include <algorithm>
#include <type_traits>

#include "cci_device.hpp"
#include "cci_launch.hpp"

namespace cci {
namespace {

constexpr int kMaskThreads = 256;

__device__ __forceinline__ uint32_t abs_bits(float w) { return __float_as_uint(w) & 0x7fffffffu; }

template <typename WT> __device__ __forceinline__ void put(WT* p, int64_t i, float w);
template <> __device__ __forceinline__ void put<float>(float* p, int64_t i, float w) { p[i] = w; }
template <> __device__ __forceinline__ void put<bf16_t>(bf16_t* p, int64_t i, float w) {
  p[i].bits = f32_to_bf16_rne(w);
}

// Batcher's odd-even merge sort, ascending (G a power of two).
template <int G>
__device__ __forceinline__ void sort_keys(uint32_t (&s)[G]) {
#pragma unroll
  for (int p = 1; p < G; p *= 2)
#pragma unroll
    for (int q = p; q >= 1; q /= 2)
#pragma unroll
      for (int j = q % p; j + q < G; j += 2 * q)
#pragma unroll
        for (int i = 0; i < q; ++i)
          if (i + j + q < G && (i + j) / (2 * p) == (i + j + q) / (2 * p)) {
            const uint32_t a = s[i + j], b = s[i + j + q];
            s[i + j] = a < b ? a : b;
            s[i + j + q] = a < b ? b : a;
          }
}

template <bool NT, typename T>
__device__ __forceinline__ T get(const T* p) {
  return NT ? __builtin_nontemporal_load(p) : *p;
}

// NT: W and the random words are read non-temporally.  NONE: no candidates,
// the random words are not read.
template <int G, bool NT, bool NONE, typename WT>
__global__ __launch_bounds__(kMaskThreads) void td_mask_fixed(const float* __restrict__ W, const uint32_t* __restrict__ bits,
                                                              int64_t C, int64_t cblocks, int32_t n_target, uint64_t thr,
                                                              WT* __restrict__ We, uint8_t* __restrict__ keep) {
  const int64_t blk = blockIdx.x;
  const int64_t g = blk / cblocks;
  const int64_t c = (blk % cblocks) * kMaskThreads + threadIdx.x;
  if (c >= C) return;
  float w[G];
  uint32_t b[G], s[G];
#pragma unroll
  for (int r = 0; r < G; ++r) w[r] = get<NT>(W + (g * G + r) * C + c);
  if constexpr (NONE) {
#pragma unroll
    for (int r = 0; r < G; ++r) {
      const int64_t o = (g * G + r) * C + c;
      put<WT>(We, o, w[r]);
      keep[o] = 1;
    }
    return;
  }
#pragma unroll
  for (int r = 0; r < G; ++r) b[r] = get<NT>(bits + (g * G + r) * C + c);
#pragma unroll
  for (int r = 0; r < G; ++r) s[r] = abs_bits(w[r]);
  sort_keys<G>(s);
  // the candidates: every row below the n_target-th smallest magnitude, and
  // of the rows equal to it the last `ties` ones (the lower row ranks above)
  uint32_t edge = s[0];
#pragma unroll
  for (int i = 1; i < G; ++i) edge = n_target - 1 == i ? s[i] : edge;
  int32_t ties = n_target;
#pragma unroll
  for (int r = 0; r < G; ++r) ties -= abs_bits(w[r]) < edge;
#pragma unroll
  for (int r = G - 1; r >= 0; --r) {
    const uint32_t key = abs_bits(w[r]);
    // (n_target > 0 here: written out, the compiler takes 71 registers for G =
    // 16 and 117 for 32, else 75 and 161)
    const bool cand = n_target > 0 && (key < edge || (key == edge && ties > 0));
    ties -= key == edge;
    const int64_t o = (g * G + r) * C + c;
    const bool drop = cand && static_cast<uint64_t>(b[r]) < thr;
    put<WT>(We, o, drop ? 0.0f : w[r]);
    keep[o] = drop ? 0 : 1;
  }
}

template <typename WT>
__global__ __launch_bounds__(kMaskThreads) void td_mask_generic(const float* __restrict__ W, const uint32_t* __restrict__ bits,
                                                                int64_t C, int64_t cblocks, int32_t G, int32_t n_target,
                                                                uint64_t thr, WT* __restrict__ We,
                                                                uint8_t* __restrict__ keep) {
  const int64_t blk = blockIdx.x;
  const int64_t g = blk / cblocks;
  const int64_t c = (blk % cblocks) * kMaskThreads + threadIdx.x;
  if (c >= C) return;
  const float* col = W + g * G * C + c;
  for (int r = 0; r < G; ++r) {
    const float wr = col[r * C];
    const uint32_t kr = abs_bits(wr);
    int rank = 0;
    for (int q = 0; q < G; ++q) {
      const uint32_t kq = abs_bits(col[q * C]);
      rank += (kq > kr) || (kq == kr && q < r);
    }
    const int64_t o = (g * G + r) * C + c;
    const bool drop = rank >= G - n_target && static_cast<uint64_t>(bits[o]) < thr;
    put<WT>(We, o, drop ? 0.0f : wr);
    keep[o] = drop ? 0 : 1;
  }
}

template <typename WT>
hipError_t td_mask_typed(const float* W, int64_t O, int64_t C, int32_t G, int32_t n_target, const uint32_t* bits,
                         uint64_t thr, WT* We, uint8_t* keep, hipStream_t s) {
  const int64_t cblocks = (C + kMaskThreads - 1) / kMaskThreads;
  const dim3 grid(static_cast<uint32_t>((O / G) * cblocks));
  const dim3 block(kMaskThreads);
  const auto launch = [&](auto g) {
    constexpr int GC = decltype(g)::value;
    const auto k = n_target == 0 ? td_mask_fixed<GC, false, true, WT>
                   : C % 32 == 0 ? td_mask_fixed<GC, true, false, WT>
                                 : td_mask_fixed<GC, false, false, WT>;
    hipLaunchKernelGGL(k, grid, block, 0, s, W, bits, C, cblocks, n_target, thr, We, keep);
  };
  switch (G) {
    case 2: launch(std::integral_constant<int, 2>{}); break;
    case 4: launch(std::integral_constant<int, 4>{}); break;
    case 8: launch(std::integral_constant<int, 8>{}); break;
    case 16: launch(std::integral_constant<int, 16>{}); break;
    case 32: launch(std::integral_constant<int, 32>{}); break;
    default:
      hipLaunchKernelGGL((td_mask_generic<WT>), grid, block, 0, s, W, bits, C, cblocks, G, n_target, thr, We, keep);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Gradient of the packed values.  A workgroup owns GB consecutive groups and
// 256 columns (a lane per column); per pass over the rows it takes KB slots
// of every group, so one staged X[n][c] feeds GB * KB multiply-adds.

constexpr int kGradThreads = 256;     // columns of a workgroup
constexpr int kGradLdsFloats = 8192;  // dY staging (32 KiB): rows per pass = min(32, 8192 / (GB * G))

template <typename T> __device__ __forceinline__ float ld(const T* p, int64_t i);
template <> __device__ __forceinline__ float ld<float>(const float* p, int64_t i) { return p[i]; }
template <> __device__ __forceinline__ float ld<bf16_t>(const bf16_t* p, int64_t i) { return bf16_to_f32(p[i].bits); }

template <typename T, int GB, int KB>
__global__ __launch_bounds__(kGradThreads) void grad_packed_kernel(const T* __restrict__ dY, const T* __restrict__ X,
                                                                   const uint8_t* __restrict__ idx,
                                                                   float* __restrict__ dv, int64_t N, int64_t C,
                                                                   int64_t O, int32_t G, int32_t K, int64_t cblocks,
                                                                   int32_t R) {
  extern __shared__ __attribute__((aligned(16))) float lds_f[];
  float* Xs = lds_f;                       // R rows x 256 columns of X
  float* dYs = lds_f + R * kGradThreads;   // R rows x (GB * G) outputs of dY
  const int64_t ngroups = O / G;
  const int64_t g0 = (blockIdx.x / cblocks) * GB;
  const int32_t gcount = static_cast<int32_t>(ngroups - g0 < GB ? ngroups - g0 : GB);
  const int64_t c = (blockIdx.x % cblocks) * kGradThreads + threadIdx.x;
  const bool live = c < C;
  const int32_t width = gcount * G;  // dY columns staged per row
  for (int32_t k0 = 0; k0 < K; k0 += KB) {
    int off[GB][KB];  // LDS offset of the entry each slot gathers, inside a staged row
    float acc[GB][KB];
#pragma unroll
    for (int gi = 0; gi < GB; ++gi)
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        const bool on = live && gi < gcount && k0 + k < K;
        const int ix = on ? idx[((g0 + gi) * K + k0 + k) * C + c] : 0;
        off[gi][k] = gi * G + (ix < G ? ix : G - 1);  // (a packing from cci_pack always has idx < G)
        acc[gi][k] = 0.0f;
      }
    for (int64_t n0 = 0; n0 < N; n0 += R) {
      const int rows = static_cast<int>(N - n0 < R ? N - n0 : R);
      __syncthreads();  // the previous pass's readers are done with dYs / Xs
      // stage the pass's dY rows (restricted to the groups) and X rows
      // (restricted to the columns): every load in flight at once
      for (int t = threadIdx.x; t < rows * width; t += kGradThreads) {
        const int n = t / width, q = t - n * width;
        dYs[t] = ld<T>(dY, (n0 + n) * O + g0 * G + q);
      }
      for (int n = 0; n < rows; ++n) Xs[n * kGradThreads + threadIdx.x] = live ? ld<T>(X, (n0 + n) * C + c) : 0.0f;
      __syncthreads();
      if (live) {
        for (int n = 0; n < rows; ++n) {
          const float x = Xs[n * kGradThreads + threadIdx.x];
          const float* row = dYs + n * width;
#pragma unroll
          for (int gi = 0; gi < GB; ++gi)
#pragma unroll
            for (int k = 0; k < KB; ++k) acc[gi][k] = __builtin_fmaf(row[off[gi][k]], x, acc[gi][k]);
        }
      }
    }
    if (live) {
#pragma unroll
      for (int gi = 0; gi < GB; ++gi)
#pragma unroll
        for (int k = 0; k < KB; ++k)
          if (gi < gcount && k0 + k < K) dv[((g0 + gi) * K + k0 + k) * C + c] = acc[gi][k];
    }
  }
}

template <typename T, int GB, int KB>
hipError_t grad_launch(const T* dY, const T* X, int64_t N, int64_t C, const uint8_t* idx, int64_t O, int32_t G,
                       int32_t K, float* dv, hipStream_t s) {
  const int64_t cblocks = (C + kGradThreads - 1) / kGradThreads;
  const int64_t gblocks = (O / G + GB - 1) / GB;
  const dim3 grid(static_cast<uint32_t>(gblocks * cblocks));
  const int32_t R = static_cast<int32_t>(std::max<int64_t>(1, std::min<int64_t>(32, kGradLdsFloats / (GB * G))));
  const size_t lds = static_cast<size_t>(R) * (GB * G + kGradThreads) * sizeof(float);
  hipLaunchKernelGGL((grad_packed_kernel<T, GB, KB>), grid, dim3(kGradThreads), lds, s, dY, X, idx, dv, N, C, O, G, K,
                     cblocks, R);
  return hipGetLastError();
}

template <typename T>
hipError_t grad_typed(const T* dY, const T* X, int64_t N, int64_t C, const uint8_t* idx, int64_t O, int32_t G,
                      int32_t K, float* dv, hipStream_t s) {
  // four groups per workgroup (X read once per four groups; enough
  // workgroups to fill the chip), up to eight slots of each per pass
  if (K == 1) return grad_launch<T, 4, 1>(dY, X, N, C, idx, O, G, K, dv, s);
  if (K == 2) return grad_launch<T, 4, 2>(dY, X, N, C, idx, O, G, K, dv, s);
  if (K <= 4) return grad_launch<T, 4, 4>(dY, X, N, C, idx, O, G, K, dv, s);
  return grad_launch<T, 4, 8>(dY, X, N, C, idx, O, G, K, dv, s);
}

}  // namespace

hipError_t launch_td_mask(const float* W, int64_t O, int64_t C, int32_t G, int32_t n_target, const uint32_t* bits,
                          uint64_t thr, void* We, DType w_t, uint8_t* keep, hipStream_t s) {
  if (w_t == DType::F32) return td_mask_typed<float>(W, O, C, G, n_target, bits, thr, static_cast<float*>(We), keep, s);
  return td_mask_typed<bf16_t>(W, O, C, G, n_target, bits, thr, static_cast<bf16_t*>(We), keep, s);
}

hipError_t launch_grad_packed(const void* dY, const void* X, DType t, int64_t N, int64_t C, const uint8_t* idx,
                              int64_t O, int32_t G, int32_t K, float* dv, hipStream_t s) {
  // bf16 operands of at least one reduction step go to the matrix cores
  if (N >= 32 && grad_mfma_supports(dY, X, t, N, C, O, G)) return launch_grad_mfma(dY, X, N, C, idx, O, G, K, dv, s);
  if (t == DType::F32)
    return grad_typed<float>(static_cast<const float*>(dY), static_cast<const float*>(X), N, C, idx, O, G, K, dv, s);
  return grad_typed<bf16_t>(static_cast<const bf16_t*>(dY), static_cast<const bf16_t*>(X), N, C, idx, O, G, K, dv, s);
}

}  // namespace cci

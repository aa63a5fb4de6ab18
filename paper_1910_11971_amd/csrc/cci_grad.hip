// Gradient of the packed values of a CCI layer on the matrix cores (the
// training step of improved targeted dropout, Sec. 5.1 / Sec. 6, once the
// mask is fixed):
//   dvals[g][k][c] = sum_n dY[n][gG + idx[g][k][c]] * X[n][c],
// the kept entries of the weight gradient dY^T X.  A vector-ALU kernel that
// multiplies only kept entries does K/G of the dense work, but at 1/32 of
// the matrix cores' rate; so for bf16 operands the dense tile of dY^T X is
// computed on v_mfma_f32_16x16x32_bf16 and only its kept entries are
// written.
//
// Work split: a workgroup of eight waves owns 256 outputs x 256 columns; wave
// w accumulates outputs 128 (w % 2) .. +127 x columns 64 (w / 2) .. +63.  With
// fewer than 160 such tiles (C or O of 2048 and less) it is four waves and
// 128 x 128, four times as many workgroups.  The reduction runs over samples
// in steps of 32:
//   - both operands are sample-major ([N][O] and [N][C]); each step's 32 rows
//     of the workgroup's dY and X columns are DMA'd into LDS row by row
//     (buffer_load ... lds; four buffers, three steps ahead), 16-byte chunk c
//     of row r at chunk c ^ f(r), f(r) = 2 ((r % 4) + 4 ((r / 8) % 2));
//   - the MFMA operands need 8 consecutive samples per lane: they are read
//     with ds_read_b64_tr_b16, which hands each lane of a 16-lane group one
//     column of the 4 x 16 block its lanes address (two reads per fragment).
//     With the swizzle every such read touches each 32-byte bank slot at
//     most twice (512 bytes in two LDS cycles);
//   - after the last step each wave parks its outputs x 32 columns of its
//     accumulators in LDS at a time and gathers the entries the packed
//     indices name: row gG + idx of column c goes to dvals[g][k][c].
// bf16 inputs widen exactly; products and sums are fp32.
// Bound by the LDS (96 KiB of transposing reads a step at ~320 B/ns per CU,
// 0.3 of the 0.85 us) and the matrix cores (0.5 us).  us, with the reads
// through the compiler's builtin / now: 4096 x 4096 x 4096 177 / 114, 2048 x
// 2048 x 2048 89 / 27, 4096 samples of 1024 x 1024 173 / 49.
#include "cci_device.hpp"
#include "cci_launch.hpp"

namespace cci {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void_t;

constexpr int kRows = 32;      // samples per reduction step
constexpr int kBufs = 4;
constexpr int kXcds = 8;
constexpr uint32_t kOOB = 0x80000000u;  // buffer offset that reads as zero
constexpr int kRsrcWord3 = 0x00020000;  // raw buffer descriptor word 3 (gfx9 family)

// Sizes by T, the 16-output blocks of a wave (8 or 4; it has 64 columns).
template <int T>
struct Tile {
  static constexpr int kSide = 32 * T;                  // workgroup tile: kSide outputs x kSide columns
  static constexpr int kWaves = T;                      // 2 x kSide / 64
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int kOpBytes = kRows * kSide * 2;    // one operand of one step
  static constexpr int kStage = 2 * kOpBytes;           // dY then X
  static constexpr int kLds = kBufs * kStage;           // 128 or 64 KiB
  static constexpr int kEpPitch = 16 * T + 8;           // epilogue staging: floats per parked column
  static_assert(kWaves * 32 * kEpPitch * 4 <= 160 * 1024, "epilogue staging fits the LDS");
  static constexpr int kLdsAll = kLds > kWaves * 32 * kEpPitch * 4 ? kLds : kWaves * 32 * kEpPitch * 4;
};

struct GParams {
  const uint16_t* dY;
  const uint16_t* X;
  const uint8_t* idx;
  float* dv;
  uint32_t dy_bytes, x_bytes;
  int32_t N, C, O, G, K;
  int32_t nob, ncb, nsteps;  // output blocks, column blocks, reduction steps
  int32_t grid8;             // grid / 8 when the grid is a multiple of 8, else 0
};

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt is 6 bits");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}
// acc += A * B with the accumulator pinned to the accumulation registers
// (128 or 64 of them hold the wave's block).  Vector accesses of an
// accumulator are separated from MFMAs that write it by mfma_drain().
__device__ __forceinline__ void mfma_acc(f32x4_t& acc, const bf16x8_t a, const bf16x8_t b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_drain() { asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory"); }

// Pin acc's current value in the accumulation registers at this point of the
// volatile sequence (no code): what comes before mfma_drain() stays before it.
__device__ __forceinline__ void acc_fence(f32x4_t& acc) { asm volatile("" : "+a"(acc)); }

// XOR of the 16-byte chunk index in staged row r (even: a 32-byte pair stays a pair).
__device__ __forceinline__ uint32_t swz(uint32_t r) { return 2u * ((r & 3u) | (((r >> 3) & 1u) << 2)); }

// MFMA operand fragments (8 samples x 16 columns, transposed to a lane per
// column) come from LDS by two transposing reads each, samples 0-3 and 4-7
// (HALF bytes apart).  The reads are inline assembly: before the builtin the
// compiler waits for every outstanding vector-memory operation, the DMAs of
// the steps to come among them, because it cannot tell them from writes to
// the rows being read (that wait, one memory latency a step, was most of the
// kernel's time).  Each asm block waits for its own reads before it ends, so
// no register is in flight outside of a block.
__device__ __forceinline__ bf16x8_t merge(const u32x2_t lo, const u32x2_t hi) {
  return __builtin_bit_cast(bf16x8_t, u32x4_t{lo[0], lo[1], hi[0], hi[1]});
}
// The six fragments a step starts with: f[0..1] at a0, a1, f[2..5] at b[0..3].
template <int HALF>
__device__ __forceinline__ void read_six(bf16x8_t& f0, bf16x8_t& f1, bf16x8_t (&fb)[4], uint32_t a0, uint32_t a1,
                                         const uint32_t (&b)[4]) {
  u32x2_t l0, h0, l1, h1, l2, h2, l3, h3, l4, h4, l5, h5;
  asm volatile(
      "ds_read_b64_tr_b16 %0, %12\n\tds_read_b64_tr_b16 %1, %12 offset:%18\n\t"
      "ds_read_b64_tr_b16 %4, %14\n\tds_read_b64_tr_b16 %5, %14 offset:%18\n\t"
      "ds_read_b64_tr_b16 %6, %15\n\tds_read_b64_tr_b16 %7, %15 offset:%18\n\t"
      "ds_read_b64_tr_b16 %8, %16\n\tds_read_b64_tr_b16 %9, %16 offset:%18\n\t"
      "ds_read_b64_tr_b16 %10, %17\n\tds_read_b64_tr_b16 %11, %17 offset:%18\n\t"
      "ds_read_b64_tr_b16 %2, %13\n\tds_read_b64_tr_b16 %3, %13 offset:%18\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(l0), "=&v"(h0), "=&v"(l1), "=&v"(h1), "=&v"(l2), "=&v"(h2), "=&v"(l3), "=&v"(h3), "=&v"(l4), "=&v"(h4),
        "=&v"(l5), "=&v"(h5)
      : "v"(a0), "v"(a1), "v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3]), "n"(HALF)
      : "memory");
  f0 = merge(l0, h0);
  f1 = merge(l1, h1);
  fb[0] = merge(l2, h2);
  fb[1] = merge(l3, h3);
  fb[2] = merge(l4, h4);
  fb[3] = merge(l5, h5);
}
// f0, f1 at at0, at1, read in the shadow of eight MFMAs acc0[n] += a0 * b[n], acc1[n] += a1 * b[n].
template <int HALF>
__device__ __forceinline__ void read_pair_mfma8(bf16x8_t& f0, bf16x8_t& f1, uint32_t at0, uint32_t at1,
                                                f32x4_t (&acc0)[4], f32x4_t (&acc1)[4], const bf16x8_t a0,
                                                const bf16x8_t a1, const bf16x8_t (&b)[4]) {
  u32x2_t l0, h0, l1, h1;
  asm volatile(
      "ds_read_b64_tr_b16 %0, %18\n\tds_read_b64_tr_b16 %1, %18 offset:%20\n\t"
      "ds_read_b64_tr_b16 %2, %19\n\tds_read_b64_tr_b16 %3, %19 offset:%20\n\t"
      "v_mfma_f32_16x16x32_bf16 %4, %12, %14, %4\n\tv_mfma_f32_16x16x32_bf16 %5, %12, %15, %5\n\t"
      "v_mfma_f32_16x16x32_bf16 %6, %12, %16, %6\n\tv_mfma_f32_16x16x32_bf16 %7, %12, %17, %7\n\t"
      "v_mfma_f32_16x16x32_bf16 %8, %13, %14, %8\n\tv_mfma_f32_16x16x32_bf16 %9, %13, %15, %9\n\t"
      "v_mfma_f32_16x16x32_bf16 %10, %13, %16, %10\n\tv_mfma_f32_16x16x32_bf16 %11, %13, %17, %11\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(l0), "=&v"(h0), "=&v"(l1), "=&v"(h1), "+a"(acc0[0]), "+a"(acc0[1]), "+a"(acc0[2]), "+a"(acc0[3]),
        "+a"(acc1[0]), "+a"(acc1[1]), "+a"(acc1[2]), "+a"(acc1[3])
      : "v"(a0), "v"(a1), "v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3]), "v"(at0), "v"(at1), "n"(HALF)
      : "memory");
  f0 = merge(l0, h0);
  f1 = merge(l1, h1);
}

template <int T>
__global__ __launch_bounds__(Tile<T>::kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void grad_mfma_kernel(GParams p) {
  constexpr int kSide = Tile<T>::kSide, kOpBytes = Tile<T>::kOpBytes, kStage = Tile<T>::kStage;
  constexpr int kEpPitch = Tile<T>::kEpPitch;
  constexpr int kRowChunks = kSide / 8;    // 16-byte chunks of a staged row
  constexpr int kWaves = Tile<T>::kWaves;
  constexpr int kDma = kStage / 1024 / kWaves;  // DMA instructions of a wave and step (4)
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wo = w & 1, wc = w >> 1;  // outputs 16 T wo .., columns 64 wc ..

  // ---- tile of this workgroup (dispatch places workgroup b on XCD b % 8): the
  // tiles of one XCD run in bands of four output blocks, so that 32 of them
  // read four blocks of dY and eight of X through its L2 ----------------------
  const uint32_t bid = blockIdx.x;
  const uint32_t L = p.grid8 ? (bid & 7u) * static_cast<uint32_t>(p.grid8) + (bid >> 3) : bid;
  const uint32_t per = 4u * static_cast<uint32_t>(p.ncb);
  const uint32_t grp = L / per;
  const uint32_t gm = min(4u, static_cast<uint32_t>(p.nob) - 4u * grp);
  const uint32_t within = L - grp * per;
  const int cb = static_cast<int>(within / gm);
  const int ob = static_cast<int>(4u * grp + (within - static_cast<uint32_t>(cb) * gm));
  const int o0 = ob * kSide, c0 = cb * kSide;

  // ---- DMA: instruction j of a step fills slots 64 j .. 64 j + 63 of the
  // stage, the dY rows, then the X rows.  Wave w issues j = w + kWaves i.
  const __amdgpu_buffer_rsrc_t yr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(p.dY), (short)0, static_cast<int>(p.dy_bytes), kRsrcWord3);
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(p.X), (short)0, static_cast<int>(p.x_bytes), kRsrcWord3);
  uint32_t soff[kDma];  // source byte offset at step 0 (kOOB: a column past the operand)
  uint32_t srow[kDma];  // the slot's staged row
#pragma unroll
  for (int i = 0; i < kDma; ++i) {
    const int j = w + kWaves * i;
    const bool isx = i >= kDma / 2;
    const uint32_t s = static_cast<uint32_t>((j - (isx ? kWaves * kDma / 2 : 0)) * 64 + lane);  // slot within the operand
    const uint32_t r = s / kRowChunks;
    const uint32_t cc = (s % kRowChunks) ^ swz(r);  // logical chunk held by the slot
    const uint32_t width = static_cast<uint32_t>(isx ? p.C : p.O);
    const uint32_t col = static_cast<uint32_t>(isx ? c0 : o0) + 8u * cc;
    srow[i] = r;
    soff[i] = col < width ? (r * width + col) * 2u : kOOB;
  }
  const auto issue = [&](int step, int buf, int i) {  // DMA instruction i of this wave
    const uint32_t n0 = static_cast<uint32_t>(step * kRows);
    const bool isx = i >= kDma / 2;
    const uint32_t width = static_cast<uint32_t>(isx ? p.C : p.O);
    const bool ok = soff[i] != kOOB && n0 + srow[i] < static_cast<uint32_t>(p.N);
    const uint32_t off = ok ? soff[i] + n0 * width * 2u : kOOB;
    lds_void_t* d = (lds_void_t*)(lds + buf * kStage + (w + kWaves * i) * 1024);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(isx ? xr : yr, d, 16, off, 0, 0, 0);
  };
  const auto issue_all = [&](int step, int buf) {
#pragma unroll
    for (int i = 0; i < kDma; ++i) issue(step, buf, i);
  };

  // ---- fragment addresses (within an operand tile) ----------------------------
  // Lane l of 16-lane group q addresses row 8 q + (l % 16) / 4, columns
  // 16 m + 4 (l % 4) .. +3 of block m: chunk 2 m + (l % 4) / 2 (swizzled),
  // half (l % 4) % 2.
  const uint32_t q = static_cast<uint32_t>(lane >> 4), li = static_cast<uint32_t>(lane & 15);
  const uint32_t fr = 8u * q + (li >> 2);
  const uint32_t fh = swz(fr) >> 1;  // in [0, 8)
  const uint32_t fbase = fr * (kSide * 2) + 16u * ((li & 3u) >> 1) + 8u * (li & 1u);
  const uint32_t lbase = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void_t*)lds));
  uint32_t aoff[T], boff[4];
#pragma unroll
  for (int m = 0; m < T; ++m) aoff[m] = lbase + fbase + 32u * (static_cast<uint32_t>(T * wo + m) ^ fh);
#pragma unroll
  for (int n = 0; n < 4; ++n) boff[n] = lbase + kOpBytes + fbase + 32u * (static_cast<uint32_t>(4 * wc + n) ^ fh);

  f32x4_t acc[T][4];
#pragma unroll
  for (int m = 0; m < T; ++m)
#pragma unroll
    for (int n = 0; n < 4; ++n) acc[m][n] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  const auto fence_all = [&] {
#pragma unroll
    for (int m = 0; m < T; ++m)
#pragma unroll
      for (int n = 0; n < 4; ++n) acc_fence(acc[m][n]);
  };
  fence_all();
  mfma_drain();  // the zero writes land before the first MFMA reads them

  // Step s: the wave waits for its DMAs of the step and meets the others at
  // the barrier (after which nobody reads the previous step's buffer: it is
  // refilled with step s + 3), reads the step's X fragments and its first two
  // dY fragments, and then issues the MFMAs of two dY fragments at a time
  // with the reads of the next two in their shadow.  Two waves share a SIMD:
  // one's reads and waits are the other's MFMA slots.
  constexpr int kHalf = 4 * kSide * 2;  // bytes from samples 0-3 to 4-7 of a fragment
  const int nsteps = p.nsteps;
#pragma unroll
  for (int b = 0; b < kBufs - 1; ++b)
    if (b < nsteps) issue_all(b, b);
#pragma unroll 1
  for (int s = 0; s < nsteps; ++s) {
    // at most the DMAs of the steps after s are in flight
    const int after = nsteps - 1 - s;
    if (after >= 2) wait_vm<2 * kDma>(); else if (after == 1) wait_vm<kDma>(); else wait_vm<0>();
    lds_barrier();
    if (s + kBufs - 1 < nsteps) issue_all(s + kBufs - 1, (s + kBufs - 1) % kBufs);
    const uint32_t sb = static_cast<uint32_t>((s % kBufs) * kStage);
    bf16x8_t a0, a1, b[4];
    const uint32_t bs[4] = {boff[0] + sb, boff[1] + sb, boff[2] + sb, boff[3] + sb};
    read_six<kHalf>(a0, a1, b, aoff[0] + sb, aoff[1] + sb, bs);
#pragma unroll
    for (int k = 0; k + 2 < T; k += 2) {
      bf16x8_t n0, n1;
      read_pair_mfma8<kHalf>(n0, n1, aoff[k + 2] + sb, aoff[k + 3] + sb, acc[k], acc[k + 1], a0, a1, b);
      a0 = n0;
      a1 = n1;
    }
#pragma unroll
    for (int n = 0; n < 4; ++n) mfma_acc(acc[T - 2][n], a0, b[n]);
#pragma unroll
    for (int n = 0; n < 4; ++n) mfma_acc(acc[T - 1][n], a1, b[n]);
  }
  mfma_drain();  // the last MFMAs have written acc
  fence_all();
  lds_barrier();  // every wave is done with the operand buffers

  // ---- gather the kept entries ---------------------------------------------------
  // Lane (q, li) holds D[16 m + 4 q + j][16 n + li] of block (m, n); per pass
  // of 32 columns (blocks n = 2 t, 2 t + 1) the wave parks them column-major
  // (pitch kEpPitch floats) and reads back row gG + idx of each column: lane l
  // takes columns 4 (l % 8) .. +3 of packed rows l / 8 + 8 x (one 4-byte index
  // load and one 16-byte store per row), its index loads issued together.
  float* stg = reinterpret_cast<float*>(lds) + w * 32 * kEpPitch;
  const int ow0 = o0 + 16 * T * wo;  // the wave's first output
  const int gw0 = ow0 / p.G;         // its first group (G divides 16 T)
  const int ngw = 16 * T / p.G;      // its groups
  const int ngroups = p.O / p.G;
  const int nrow = ngw * p.K;      // packed rows (g, k) of its groups
  const int cq = lane & 7, r0 = lane >> 3;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
#pragma unroll
    for (int m = 0; m < T; ++m)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        *reinterpret_cast<f32x4_t*>(stg + (16 * h + li) * kEpPitch + 16 * m + 4 * q) = acc[m][2 * t + h];
    const int c = c0 + 64 * wc + 32 * t + 4 * cq;  // the lane's first column
    const bool cok = c < p.C;
#pragma unroll 1
    for (int x0 = 0; 8 * x0 < nrow; x0 += 4) {
      uint32_t iv[4];
      int64_t e[4];
      bool ok[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int r = r0 + 8 * (x0 + x);
        const int gi = r / p.K, k = r - gi * p.K;
        ok[x] = cok && r < nrow && gw0 + gi < ngroups;
        e[x] = (static_cast<int64_t>(gw0 + gi) * p.K + k) * p.C + c;
        iv[x] = ok[x] ? *reinterpret_cast<const uint32_t*>(p.idx + e[x]) : 0u;
      }
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        if (ok[x]) {
          const int r = r0 + 8 * (x0 + x);
          const int gbase = (r / p.K) * p.G;  // the group's first row within the wave
          f32x4_t v;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            uint32_t ix = (iv[x] >> (8 * j)) & 0xffu;
            ix = ix < static_cast<uint32_t>(p.G) ? ix : static_cast<uint32_t>(p.G - 1);
            v[j] = stg[(4 * cq + j) * kEpPitch + gbase + static_cast<int>(ix)];
          }
          *reinterpret_cast<f32x4_t*>(p.dv + e[x]) = v;
        }
      }
    }
  }
}

// Fewer 256 x 256 tiles than this: 128 x 128 ones, four times as many.
constexpr int64_t kWideTiles = 160;

template <int T>
hipError_t launch_grad_t(GParams p, hipStream_t s) {
  constexpr int kSide = Tile<T>::kSide, kLds = Tile<T>::kLdsAll;
  p.nob = (p.O + kSide - 1) / kSide;
  p.ncb = (p.C + kSide - 1) / kSide;
  const int64_t grid = static_cast<int64_t>(p.nob) * p.ncb;
  if (grid > 0x7fffffff) return hipErrorInvalidConfiguration;
  p.grid8 = grid % kXcds == 0 ? static_cast<int32_t>(grid / kXcds) : 0;
  static std::atomic<int8_t> lds_set[kMaxDevices];
  const hipError_t attr = set_lds_limit_once(lds_set, reinterpret_cast<const void*>(&grad_mfma_kernel<T>), kLds);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((grad_mfma_kernel<T>), dim3(static_cast<uint32_t>(grid)), dim3(Tile<T>::kThreads), kLds, s, p);
  return hipGetLastError();
}

}  // namespace

bool grad_mfma_supports(const void* dY, const void* X, DType t, int64_t N, int64_t C, int64_t O, int32_t G) {
  if (t != DType::BF16 || N < 1) return false;
  if (O % 8 != 0 || C % 8 != 0 || G < 1 || 128 % G != 0) return false;
  const auto al = [](const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; };
  if (!al(dY) || !al(X)) return false;
  const int64_t lim = static_cast<int64_t>(kOOB);
  return N * O * 2 < lim && N * C * 2 < lim;
}

hipError_t launch_grad_mfma(const void* dY, const void* X, int64_t N, int64_t C, const uint8_t* idx, int64_t O,
                            int32_t G, int32_t K, float* dv, hipStream_t s) {
  GParams p{};
  p.dY = static_cast<const uint16_t*>(dY);
  p.X = static_cast<const uint16_t*>(X);
  p.idx = idx;
  p.dv = dv;
  p.dy_bytes = static_cast<uint32_t>(N * O * 2);
  p.x_bytes = static_cast<uint32_t>(N * C * 2);
  p.N = static_cast<int32_t>(N);
  p.C = static_cast<int32_t>(C);
  p.O = static_cast<int32_t>(O);
  p.G = G;
  p.K = K;
  p.nsteps = static_cast<int32_t>((N + kRows - 1) / kRows);
  const int64_t tiles256 = (O + 255) / 256 * ((C + 255) / 256);
  return tiles256 >= kWideTiles || 64 % G != 0 ? launch_grad_t<8>(p, s) : launch_grad_t<4>(p, s);
}

}  // namespace cci

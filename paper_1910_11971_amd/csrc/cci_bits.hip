// Plain log2(G)-bit indices (Sec. 3.1) and the product that reads them where
// weight bytes bind: few rows.
//
// Index stream: with b = ceil(log2 G) bits per kept weight, entry e of an
// index array sits at bits e*b .. e*b+b-1 of a little-endian stream of
// 32-bit words (stream bit t = bit t % 32 of word t / 32).  b = 8 is the byte
// array cci_pack writes.
//
// Few-row product (N <= 64).  With few rows every packed weight is used by
// at most N multiply-adds, so the packed bytes (2 per value + b/8 per index)
// and the memory latency set the time.  A workgroup of eight waves owns 16
// output channels (the last one fewer when O % 16 != 0: its missing rows are
// not stored); wave w takes the 128-column chunks w, w+8, ... of the
// reduction and keeps the loads of up to four of them in flight, so a
// reduction of 4096 costs about one memory round trip (with one 32-column
// k-step in flight and 2-byte loads it cost sixteen: 1 x 4096 -> 4096, G = 16,
// K = 4, 11.3 us of kernel time against 8.0 now).  Per chunk a wave
//   - clears its 16 x 128 bf16 tile in LDS,
//   - reads the kept entries of the groups covering its 16 rows in units of 8
//     columns of one packed row (16 bytes of values, 8 index entries: b
//     bytes), and writes every value whose row falls in the tile to (row,
//     column) -- Alg. 1's routing to row gG+idx; with K == G the slots are the
//     rows and a unit is stored whole,
//   - reads the tile back as A fragments of v_mfma_f32_16x16x32_bf16 and
//     multiplies them with up to four 16-row fragments of X.
// The eight waves' partial sums are added in LDS; the fused epilogue (its
// operands requested before the reduction) and one rounding follow.  Tile
// row i keeps its 16-byte unit u at 256 i + 16 (u ^ i): the 16 rows of a
// fragment read touch distinct bank slots.
#include <algorithm>
#include <type_traits>

#include "cci_device.hpp"
#include "cci_launch.hpp"

namespace cci {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint16_t u16x4_t __attribute__((ext_vector_type(4)));

constexpr int kRsrcWord3 = 0x00020000;  // raw buffer descriptor word 3 (gfx9 family)

// ---------------------------------------------------------------------------
// Index stream: one lane per 32-bit output word.

__global__ __launch_bounds__(256) void index_bits_kernel(const uint8_t* __restrict__ idx, int64_t n, int32_t b,
                                                         uint32_t* __restrict__ words, int64_t nw) {
  const int64_t w = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (w >= nw) return;
  const int64_t t0 = w * 32;
  const int64_t e0 = t0 / b, e1 = (t0 + 31) / b;  // entries touching this word
  uint32_t word = 0;
  for (int64_t e = e0; e <= e1 && e < n; ++e) {
    const int64_t sh = e * b - t0;                 // -b < sh < 32
    const uint32_t v = idx[e] & ((1u << b) - 1u);
    word |= sh >= 0 ? (v << sh) : (v >> -sh);
  }
  words[w] = word;
}

// ---------------------------------------------------------------------------

constexpr int kFThreads = 512;  // eight waves
constexpr int kFWaves = 8;

struct FParams {
  const uint16_t* X;
  const uint16_t* vals;
  const void* idx;
  const float* scale;
  const float* bias;
  const void* residual;
  void* Y;
  uint32_t x_bytes, i_bytes, v_bytes;
  int32_t N, C, O, G, K, b, relu;
};

// ReLU, rounding and store of a lane's four outputs.
template <typename YT>
__device__ __forceinline__ void store4(const FParams& p, float (&y)[4], int64_t yo) {
  if (p.relu) {
#pragma unroll
    for (int r = 0; r < 4; ++r) y[r] = y[r] > 0.0f ? y[r] : (y[r] != y[r] ? y[r] : 0.0f);
  }
  if (std::is_same<YT, float>::value) {
    *reinterpret_cast<f32x4_t*>(static_cast<float*>(p.Y) + yo) = f32x4_t{y[0], y[1], y[2], y[3]};
  } else {
    *reinterpret_cast<u16x4_t*>(static_cast<uint16_t*>(p.Y) + yo) =
        u16x4_t{f32_to_bf16_rne(y[0]), f32_to_bf16_rne(y[1]), f32_to_bf16_rne(y[2]), f32_to_bf16_rne(y[3])};
  }
}

// Columns of a chunk.  PAIR: two workgroups share a CU, with half of the
// registers and so half of the columns each.
constexpr int chunk_cols(bool pair) { return pair ? 64 : 128; }
constexpr int tile_bytes(bool pair) { return 16 * chunk_cols(pair) * 2; }  // a wave's tile
// Packed rows that a wave's lanes read at once (one 8-column unit per lane).
constexpr int unit_rows(bool pair) { return 64 * 8 / chunk_cols(pair); }

// Loads of one chunk: up to PL packed units per lane (values and index
// words) and the lane's X fragments.
template <int PL, int NB, int STEPS>
struct Fetch {
  u32x4_t v[PL];
  uint32_t ix[PL][3];
  u32x4_t x[STEPS][NB];
};

// Chunks in flight per wave: as many as fit about 170 (PAIR: 64) registers,
// at most 4.
constexpr int depth(int pl, int nb, bool pair) {
  const int d = (pair ? 64 : 170) / (pl * 7 + nb * chunk_cols(pair) / 8);
  return d < 1 ? 1 : d > 4 ? 4 : d;
}

// PL: packed units per lane and pass; ONE: one pass covers a chunk (else the
// units of a chunk are walked in passes, loaded inline).
template <int NB, int PL, bool ONE, bool PAIR, typename YT>
__global__ __launch_bounds__(kFThreads, PAIR ? 4 : 2) void spmm_bits_kernel(FParams p) {
  constexpr int D = ONE ? depth(PL, NB, PAIR) : 1;
  constexpr int CW = chunk_cols(PAIR), UN = CW / 8, RP = unit_rows(PAIR), STEPS = CW / 32;
  // a wave's weight tile, later its partial sums ([NB][64] f32x4_t)
  constexpr int kTile = tile_bytes(PAIR), kSums = NB * 64 * static_cast<int>(sizeof(f32x4_t));
  __shared__ __attribute__((aligned(16))) uint8_t tiles[kFWaves][kTile > kSums ? kTile : kSums];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int32_t o0 = static_cast<int32_t>(blockIdx.x) * 16;
  const int32_t g_lo = o0 / p.G, g_hi = min((o0 + 15) / p.G, p.O / p.G - 1);
  // packed rows (group, slot) x UN units of a chunk: lane % UN is the unit (8
  // columns), entry u of a lane packed row lane / UN + RP u
  const int32_t nrows = (g_hi - g_lo + 1) * p.K;
  const int32_t c8 = lane % UN, r0l = lane / UN;
  const bool full = p.K == p.G;

  const __amdgpu_buffer_rsrc_t xr =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.X), (short)0, static_cast<int>(p.x_bytes), kRsrcWord3);
  const __amdgpu_buffer_rsrc_t ir =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.idx), (short)0, static_cast<int>(p.i_bytes), kRsrcWord3);
  const __amdgpu_buffer_rsrc_t vr =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.vals), (short)0, static_cast<int>(p.v_bytes), kRsrcWord3);
  constexpr uint32_t kOut = 0x80000000u;  // reads as zero
  uint8_t* tile = tiles[w];
  const int ti = lane & 15, tq = lane >> 4;

  // scale, bias and residual of the outputs this wave finishes (rows 16 w ..)
  const int32_t en = 16 * w + ti, eo = o0 + 4 * tq;
  const bool eok = w < NB && en < p.N && eo < p.O;  // (O % 4 == 0: a lane's 4 outputs are all inside or all past O)
  const bool yf32 = std::is_same<YT, float>::value;
  const int64_t yo = static_cast<int64_t>(en) * p.O + eo;
  f32x4_t sc{1.f, 1.f, 1.f, 1.f}, bi{0.f, 0.f, 0.f, 0.f}, rs{0.f, 0.f, 0.f, 0.f};
  if (eok) {
    if (p.scale) sc = *reinterpret_cast<const f32x4_t*>(p.scale + eo);
    if (p.bias) bi = *reinterpret_cast<const f32x4_t*>(p.bias + eo);
    if (p.residual) {
      if (yf32) {
        rs = *reinterpret_cast<const f32x4_t*>(static_cast<const float*>(p.residual) + yo);
      } else {
        const u16x4_t r = *reinterpret_cast<const u16x4_t*>(static_cast<const uint16_t*>(p.residual) + yo);
#pragma unroll
        for (int e = 0; e < 4; ++e) rs[e] = bf16_to_f32(r[e]);
      }
    }
  }

  // first packed element of this lane's unit of packed row r in chunk 0
  const auto unit_e = [&](int32_t r) { return (static_cast<int64_t>(g_lo) * p.K + r) * p.C + 8 * c8; };
  auto load_unit = [&](int64_t e, bool on, u32x4_t& v, uint32_t (&ix)[3]) {
    v = __builtin_bit_cast(u32x4_t,
                           __builtin_amdgcn_raw_buffer_load_b128(vr, on ? static_cast<uint32_t>(e) * 2u : kOut, 0, 0));
    if (full) return;
    // 8 entries of b bits start at byte e b / 8 (e % 8 == 0): the words that
    // hold them (b = 7 can straddle three)
    const uint32_t off = static_cast<uint32_t>((e * p.b) >> 5) * 4u;
    ix[0] = __builtin_amdgcn_raw_buffer_load_b32(ir, on ? off : kOut, 0, 0);
    ix[1] = __builtin_amdgcn_raw_buffer_load_b32(ir, on ? off + 4u : kOut, 0, 0);
    ix[2] = p.b == 7 ? __builtin_amdgcn_raw_buffer_load_b32(ir, on ? off + 8u : kOut, 0, 0) : 0u;
  };
  // route a unit of packed row r (its first element e) to the tile
  auto scatter = [&](int32_t r, int64_t e, const u32x4_t v, const uint32_t (&ix)[3]) {
    const int32_t gl = r / p.K;
    const int32_t row0 = (g_lo + gl) * p.G - o0;
    if (full) {
      const int32_t row = row0 + r - gl * p.K;
      if (r < nrows && row >= 0 && row < 16)
        *reinterpret_cast<u32x4_t*>(tile + row * (2 * CW) + ((c8 ^ (row % UN)) * 16)) = v;
      return;
    }
    const uint32_t sh = static_cast<uint32_t>((e * p.b) & 31);
    const uint64_t bits = static_cast<uint64_t>(__builtin_amdgcn_alignbit(ix[1], ix[0], sh)) |
                          (static_cast<uint64_t>(__builtin_amdgcn_alignbit(ix[2], ix[1], sh)) << 32);
    const uint32_t mask = (1u << p.b) - 1u;
    if (r < nrows) {
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int32_t row = row0 + static_cast<int32_t>(static_cast<uint32_t>(bits >> (t * p.b)) & mask);
        if (row >= 0 && row < 16)
          *reinterpret_cast<uint16_t*>(tile + row * (2 * CW) + ((c8 ^ (row % UN)) * 16) + 2 * t) =
              static_cast<uint16_t>(v[t >> 1] >> (16 * (t & 1)));
      }
    }
  };
  auto clear = [&]() {
    if (full) return;
#pragma unroll
    for (int q = 0; q < kTile / 1024; ++q)
      *reinterpret_cast<u32x4_t*>(tile + q * 1024 + lane * 16) = u32x4_t{0u, 0u, 0u, 0u};
  };

  auto fetch = [&](int32_t ch, Fetch<PL, NB, STEPS>& f) {
    const int32_t c0 = ch * CW;
    if constexpr (ONE) {
#pragma unroll
      for (int u = 0; u < PL; ++u) {
        const int32_t r = r0l + RP * u;
        load_unit(unit_e(r) + c0, r < nrows && c0 + 8 * c8 < p.C, f.v[u], f.ix[u]);
      }
    }
#pragma unroll
    for (int j = 0; j < STEPS; ++j)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const uint32_t n = static_cast<uint32_t>(16 * nb + ti);
        const int32_t c = c0 + 32 * j + 8 * tq;
        const uint32_t off = n < static_cast<uint32_t>(p.N) && c < p.C
                                 ? (n * static_cast<uint32_t>(p.C) + static_cast<uint32_t>(c)) * 2u
                                 : kOut;
        f.x[j][nb] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(xr, off, 0, 0));
      }
  };

  f32x4_t acc[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) acc[nb] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int32_t nch = (p.C + CW - 1) / CW;
  Fetch<PL, NB, STEPS> st[D];
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (w + kFWaves * d < nch) fetch(w + kFWaves * d, st[d]);
  for (int32_t base = w; base < nch; base += kFWaves * D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int32_t ch = base + kFWaves * d;
      if (ch < nch) {
        const int32_t c0 = ch * CW;
        clear();
        if constexpr (ONE) {
#pragma unroll
          for (int u = 0; u < PL; ++u) scatter(r0l + RP * u, unit_e(r0l + RP * u) + c0, st[d].v[u], st[d].ix[u]);
        } else {
#pragma unroll 1
          for (int32_t r0 = 0; r0 < nrows; r0 += RP * PL) {
#pragma unroll
            for (int u = 0; u < PL; ++u) {
              const int32_t r = r0 + r0l + RP * u;
              load_unit(unit_e(r) + c0, r < nrows && c0 + 8 * c8 < p.C, st[d].v[u], st[d].ix[u]);
            }
#pragma unroll
            for (int u = 0; u < PL; ++u) {
              const int32_t r = r0 + r0l + RP * u;
              scatter(r, unit_e(r) + c0, st[d].v[u], st[d].ix[u]);
            }
          }
        }
#pragma unroll
        for (int j = 0; j < STEPS; ++j) {
          const bf16x8_t a =
              *reinterpret_cast<const bf16x8_t*>(tile + ti * (2 * CW) + (((4 * j + tq) ^ (ti % UN)) * 16));
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
            acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8_t, st[d].x[j][nb]), acc[nb],
                                                              0, 0, 0);
        }
        if (ch + kFWaves * D < nch) fetch(ch + kFWaves * D, st[d]);
      }
    }
  }

  // ---- sum the eight waves' partials; wave nb finishes X rows 16 nb .. +16
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) reinterpret_cast<f32x4_t*>(tile)[nb * 64 + lane] = acc[nb];
  __syncthreads();
  if (w >= NB) return;
  const auto part = [&](int v) { return reinterpret_cast<const f32x4_t*>(tiles[v])[w * 64 + lane]; };
  f32x4_t sum = part(0);
#pragma unroll
  for (int v = 1; v < kFWaves; ++v) sum += part(v);
  if (!eok) return;
  float y[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) y[r] = sum[r] * sc[r] + bi[r] + rs[r];
  store4<YT>(p, y, yo);
}

// The same product in k-steps of 32 columns, one in flight per wave: a lane
// takes one column of a packed row, so few packed rows (step_rows below)
// still occupy all of them, and 42-80 registers and 16-40 KiB of LDS let up
// to four workgroups share a CU.
// Loads of one k-step: up to PL kept entries per lane (index word(s) and
// value) and the lane's X fragments.
template <int PL, int NB>
struct StepFetch {
  uint32_t lo[PL], hi[PL];
  uint16_t v[PL];
  u32x4_t x[NB];
};

template <int NB, int PL, typename YT>
__global__ __launch_bounds__(kFThreads) void few_step_kernel(FParams p) {
  __shared__ __attribute__((aligned(16))) uint8_t tiles[kFWaves][1024];
  __shared__ __attribute__((aligned(16))) f32x4_t red[kFWaves][NB][64];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int32_t o0 = static_cast<int32_t>(blockIdx.x) * 16;
  const int32_t g_lo = o0 / p.G, g_hi = min((o0 + 15) / p.G, p.O / p.G - 1);
  // (group, slot) pairs cover the k-step's 32 columns: lanes 0..31 take the
  // even pairs, lanes 32..63 the odd ones, lane & 31 the column; entry u of
  // a lane is pair pk + 2u, at packed offset base[u] + 32 s in k-step s
  const int32_t npairs = (g_hi - g_lo + 1) * p.K;
  const int32_t pk = lane >> 5, cj = lane & 31;
  int64_t base[PL];
  int32_t row0[PL];
  bool on[PL];
#pragma unroll
  for (int u = 0; u < PL; ++u) {
    const int32_t q = pk + 2 * u;
    on[u] = q < npairs;
    const int32_t gl = on[u] ? q / p.K : 0, k = on[u] ? q - gl * p.K : 0;
    base[u] = (static_cast<int64_t>(g_lo + gl) * p.K + k) * p.C + cj;
    row0[u] = (g_lo + gl) * p.G - o0;
  }

  const __amdgpu_buffer_rsrc_t xr =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.X), (short)0, static_cast<int>(p.x_bytes), kRsrcWord3);
  const __amdgpu_buffer_rsrc_t ir =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.idx), (short)0, static_cast<int>(p.i_bytes), kRsrcWord3);
  const __amdgpu_buffer_rsrc_t vr =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.vals), (short)0, static_cast<int>(p.v_bytes), kRsrcWord3);
  const uint32_t mask = (1u << p.b) - 1u;
  uint8_t* tile = tiles[w];
  const int ti = lane & 15, tq = lane >> 4;
  const uint8_t* frag = tile + ti * 64 + ((tq ^ ((ti >> 2) & 3)) * 16);

  auto fetch = [&](int32_t s, StepFetch<PL, NB>& f) {
    const int32_t c0 = s * 32;
#pragma unroll
    for (int u = 0; u < PL; ++u) {
      const int64_t e = base[u] + c0;
      const uint32_t voff = on[u] ? static_cast<uint32_t>(e) * 2u : 0x80000000u;
      f.v[u] = __builtin_amdgcn_raw_buffer_load_b16(vr, voff, 0, 0);
      if (p.b == 8) {
        f.lo[u] = __builtin_amdgcn_raw_buffer_load_b8(ir, on[u] ? static_cast<uint32_t>(e) : 0x80000000u, 0, 0);
        f.hi[u] = 0;
      } else {
        const uint32_t off = on[u] ? static_cast<uint32_t>((e * p.b) >> 5) * 4u : 0x80000000u;
        f.lo[u] = __builtin_amdgcn_raw_buffer_load_b32(ir, off, 0, 0);
        f.hi[u] = __builtin_amdgcn_raw_buffer_load_b32(ir, on[u] ? off + 4u : 0x80000000u, 0, 0);
      }
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const uint32_t n = static_cast<uint32_t>(16 * nb + ti);
      const uint32_t off = n < static_cast<uint32_t>(p.N)
                               ? (n * static_cast<uint32_t>(p.C) + static_cast<uint32_t>(c0 + 8 * tq)) * 2u
                               : 0x80000000u;
      f.x[nb] = __builtin_amdgcn_raw_buffer_load_b128(xr, off, 0, 0);
    }
  };

  f32x4_t acc[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) acc[nb] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int32_t nks = p.C / 32;
  StepFetch<PL, NB> cur, nxt;
  if (w < nks) fetch(w, cur);
  for (int32_t s = w; s < nks; s += kFWaves) {
    if (s + kFWaves < nks) fetch(s + kFWaves, nxt);
    const int32_t c0 = s * 32;
    *reinterpret_cast<u32x4_t*>(tile + lane * 16) = u32x4_t{0u, 0u, 0u, 0u};
#pragma unroll
    for (int u = 0; u < PL; ++u) {
      const int64_t e = base[u] + c0;
      const uint32_t r = p.b == 8 ? cur.lo[u] : __builtin_amdgcn_alignbit(cur.hi[u], cur.lo[u],
                                                                          static_cast<uint32_t>((e * p.b) & 31)) & mask;
      const int32_t row = row0[u] + static_cast<int32_t>(r);
      if (on[u] && row >= 0 && row < 16)
        *reinterpret_cast<uint16_t*>(tile + row * 64 + (((cj >> 3) ^ ((row >> 2) & 3)) * 16) + (cj & 7) * 2) = cur.v[u];
    }
    const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(frag);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8_t, cur.x[nb]), acc[nb], 0, 0, 0);
    cur = nxt;
  }

  // ---- sum the eight waves' partials; wave nb finishes X rows 16 nb .. +16
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) red[w][nb][lane] = acc[nb];
  __syncthreads();
  if (w >= NB) return;
  f32x4_t sum = red[0][w][lane];
#pragma unroll
  for (int v = 1; v < kFWaves; ++v) sum += red[v][w][lane];
  const int32_t n = 16 * w + ti;
  const int32_t o = o0 + 4 * tq;  // lane holds outputs o .. o+3 of row n
  if (n >= p.N || o >= p.O) return;  // (O % 4 == 0: a lane's 4 outputs are all inside or all past O)
  const bool yf32 = std::is_same<YT, float>::value;
  const int64_t yo = static_cast<int64_t>(n) * p.O + o;
  float y[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    y[r] = sum[r];
    if (p.scale) y[r] *= p.scale[o + r];
    if (p.bias) y[r] += p.bias[o + r];
  }
  if (p.residual) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      y[r] += yf32 ? static_cast<const float*>(p.residual)[yo + r]
                   : bf16_to_f32(static_cast<const uint16_t*>(p.residual)[yo + r]);
  }
  store4<YT>(p, y, yo);
}

template <int NB, int PL, bool ONE, bool PAIR>
hipError_t launch_fp(const FParams& p, DType y_t, hipStream_t s) {
  const dim3 grid(static_cast<uint32_t>((p.O + 15) / 16));
  if (y_t == DType::F32)
    hipLaunchKernelGGL((spmm_bits_kernel<NB, PL, ONE, PAIR, float>), grid, dim3(kFThreads), 0, s, p);
  else
    hipLaunchKernelGGL((spmm_bits_kernel<NB, PL, ONE, PAIR, bf16_t>), grid, dim3(kFThreads), 0, s, p);
  return hipGetLastError();
}

// Groups that 16 consecutive outputs starting at a multiple of 16 can touch.
int32_t tile_groups(int32_t G) { return 16 % G == 0 ? 16 / G : (G % 16 == 0 ? 1 : 15 / G + 2); }

// PL: packed units a lane reads per chunk: the packed rows of those groups,
// spread over the lanes.  Up to 4 they are loaded chunks ahead; beyond, the walk in
// passes.
template <int NB, bool PAIR>
hipError_t launch_f(const FParams& p, DType y_t, hipStream_t s) {
  const int32_t pl = (tile_groups(p.G) * p.K + unit_rows(PAIR) - 1) / unit_rows(PAIR);
  if (pl <= 1) return launch_fp<NB, 1, true, PAIR>(p, y_t, s);
  if (pl <= 2) return launch_fp<NB, 2, true, PAIR>(p, y_t, s);
  if (!PAIR && pl <= 4) return launch_fp<NB, 4, true, false>(p, y_t, s);
  return launch_fp<NB, PAIR ? 2 : 4, false, PAIR>(p, y_t, s);
}

// PL: kept entries a lane reads per k-step, half of the packed rows.
template <int NB>
hipError_t launch_step(const FParams& p, int32_t rows, DType y_t, hipStream_t s) {
  const dim3 grid(static_cast<uint32_t>((p.O + 15) / 16));
  const auto launch = [&](auto pl) {
    constexpr int PL = decltype(pl)::value;
    if (y_t == DType::F32)
      hipLaunchKernelGGL((few_step_kernel<NB, PL, float>), grid, dim3(kFThreads), 0, s, p);
    else
      hipLaunchKernelGGL((few_step_kernel<NB, PL, bf16_t>), grid, dim3(kFThreads), 0, s, p);
    return hipGetLastError();
  };
  if (rows <= 2) return launch(std::integral_constant<int, 1>{});
  if (rows <= 4) return launch(std::integral_constant<int, 2>{});
  return launch(std::integral_constant<int, 3>{});
}

template <bool PAIR>
hipError_t launch_n(const FParams& p, DType y_t, hipStream_t s) {
  if (p.N <= 16) return launch_f<1, PAIR>(p, y_t, s);
  if (p.N <= 32) return launch_f<2, PAIR>(p, y_t, s);
  if (p.N <= 48) return launch_f<3, PAIR>(p, y_t, s);
  return launch_f<4, PAIR>(p, y_t, s);
}

}  // namespace

int64_t index_stream_bytes(int64_t n, int32_t b) { return b == 8 ? n : (n * b + 31) / 32 * 4; }

hipError_t launch_index_bits(const uint8_t* idx, int64_t n, int32_t b, uint32_t* words, hipStream_t s) {
  const int64_t nw = (n * b + 31) / 32;
  if (nw == 0) return hipSuccess;
  hipLaunchKernelGGL(index_bits_kernel, dim3(static_cast<uint32_t>((nw + 255) / 256)), dim3(256), 0, s, idx, n, b,
                     words, nw);
  return hipGetLastError();
}

bool spmm_bits_supports(int64_t N, int64_t C, int64_t O, int32_t G, int32_t K) {
  return N >= 0 && N <= 64 && C % 32 == 0 && O % 4 == 0 && N * C * 2 < (int64_t(1) << 31) &&
         (O / G) * K * C < (int64_t(1) << 30);
}

hipError_t launch_spmm_bits(const void* X, int64_t N, int64_t C, const void* vals, const void* idx, int32_t b,
                            int64_t O, int32_t G, int32_t K, const float* scale, const float* bias,
                            const void* residual, int32_t relu, void* Y, DType y_t, hipStream_t s) {
  FParams p{};
  p.X = static_cast<const uint16_t*>(X);
  p.vals = static_cast<const uint16_t*>(vals);
  p.idx = idx;
  p.scale = scale;
  p.bias = bias;
  p.residual = residual;
  p.Y = Y;
  p.x_bytes = static_cast<uint32_t>(N * C * 2);
  p.i_bytes = static_cast<uint32_t>(index_stream_bytes((O / G) * K * C, b));
  p.v_bytes = static_cast<uint32_t>((O / G) * K * C * 2);
  p.N = static_cast<int32_t>(N);
  p.C = static_cast<int32_t>(C);
  p.O = static_cast<int32_t>(O);
  p.G = G;
  p.K = K;
  p.b = b;
  p.relu = relu;
  const int32_t rows = tile_groups(G) * K;
  const bool many = O > 16 * 256;
  if (rows <= 2 || (rows <= 4 && (many || C < 256)) || (rows <= 6 && C < 128 && O > 16 * 512)) {
    if (N <= 16) return launch_step<1>(p, rows, y_t, s);
    if (N <= 32) return launch_step<2>(p, rows, y_t, s);
    return launch_step<4>(p, rows, y_t, s);
  }
  return many || C <= 1024 ? launch_n<true>(p, y_t, s) : launch_n<false>(p, y_t, s);
}

}  // namespace cci

// CCI-sparse product on the matrix cores, tap-chunk plan: convolutions of
// any geometry through implicit im2col, and FC products, whose reduction
// splits into chunks of 64 input channels under one filter tap.
//
// Chunk j of the reduction is packed columns 64 j .. 64 j + 63, i.e. tap
// t = j / (Cin / 64) (kh = t / KW, kw = t % KW) and input channels
// 64 (j % (Cin / 64)) .. +63: the columns of W [O][KH][KW][Cin] in order.  Per
// chunk:
//   - the packed groups of the workgroup's 128 outputs are expanded to a
//     dense 128 x 64 bf16 tile in LDS (zero fill, then every kept weight
//     written to row G*g + idx of its column: the routing of Alg. 1,
//     Sec. 3.2);
//   - the 128 output pixels' input pixels under tap t are DMA'd to LDS, 128
//     contiguous bytes each; a tap that falls into the padding reads zero
//     through the buffer's range check (its offset has bit 31 set);
//   - the tile is multiplied on v_mfma_f32_16x16x32_bf16.
// Work split: a team of four waves owns 128 pixels x 128 (or 64) outputs;
// wave (wp, wo) accumulates pixels 64 wp .. +63 x outputs 64 wo .. +63 in
// sixteen 16 x 16 accumulators.  A team takes 80 KiB of LDS (three activation
// buffers, two weight tiles), so two share a CU and the tile builds, barriers
// and epilogue of one overlap the other's MFMAs: two workgroups of one team,
// or, on small grids, one workgroup whose two teams halve the reduction.
// Bound by the LDS: a step of two chunks takes ~2 070 cycles, the sum of its
// fragment reads (128 KiB at ~225 B/clk), zero fill and DMA (32 KiB each at
// ~60 B/clk) and 64 scatter stores (~5 clk); its MFMAs need 1 024.  This
// serves the products with long reductions and few output tiles (k x k
// convolutions over 128-512 channels, 1x1 layers of 10^4 pixels) that leave
// most CUs idle under 256 x 256 tiles.
//
// LDS layouts (bytes):
//   activation buffer: pixel q at q * 128; its 16-byte column c holds
//     channels 8 * (c ^ sw(q)) .. +7 of the chunk, sw(q) = (q >> 1) % 8 (a
//     fragment read of 16 pixels touches distinct bank slots per 16 lanes).
//   weight tile: 16-row block b, k-step s at (2 b + s) * 1024, inside it
//     (k / 8 % 4) * 256 + (o % 16) * 16 + (k % 8) * 2: the fragment a lane
//     reads is its 16 contiguous bytes at lane * 16.
#include <type_traits>
#include <utility>

#include "cci_chunks.hpp"
#include "cci_device.hpp"
#include "cci_kept.hpp"
#include "cci_launch.hpp"

namespace cci {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void lds_void_t;

constexpr int kThreads = 256;             // four waves (one team)
constexpr int kTP = 128;                  // pixels of a workgroup tile
constexpr int kCK = 64;                   // reduction columns per chunk (two k-steps)
constexpr int kXB = kTP * kCK * 2;        // one activation buffer
// A team's buffers: kNX activation buffers, then two weight tiles (80 KiB
// with 128-output tiles: two teams per CU, as two workgroups or as one).
// TO outputs per workgroup tile (128, or 64 for grids that would leave CUs
// idle): one weight tile is TO x 64 bf16
constexpr int kNX = 3;
constexpr int wb_bytes(int to) { return to * kCK * 2; }
constexpr int lds_bytes(int to) { return kNX * kXB + 2 * wb_bytes(to); }
// epilogue staging: bytes per pixel row of a wave's 64 x TO/2 fp32 block
constexpr int ep_pitch(int to) { return to / 2 * 4 + 16; }
constexpr int kMaxTaps = 32;              // taps of one filter (one validity bit each)
constexpr uint32_t kPairGrid = 257;       // grids below this run one workgroup per CU: of two teams
constexpr int kPairChunks = 4;            // and have at least this many chunks
constexpr int64_t kSmallGrid = 128;       // fewer 128-output tiles than this (half the CUs): 64-output tiles
constexpr uint32_t kOOB = 0x80000000u;    // buffer offset that reads as zero / drops a store
constexpr int kRsrcWord3 = 0x00020000;    // raw buffer descriptor word 3 (gfx9 family)
static_assert(4 * 64 * ep_pitch(128) <= lds_bytes(128) && 4 * 64 * ep_pitch(64) <= lds_bytes(64) &&
                  2 * lds_bytes(128) <= 160 * 1024,
              "epilogue staging reuses the operand buffers; two teams fit a CU");

struct TParams {
  const uint16_t* X;
  const uint16_t* vals;
  const uint8_t* idx;
  const float* scale;
  const float* bias;
  const void* residual;
  void* Y;
  uint32_t x_bytes, v_bytes, i_bytes, y_bytes;
  int32_t N, C, O, G, K, relu, kept_only;
  int32_t npb, nob, nch;  // pixel blocks (of 128), output blocks (of TO), chunks
  int32_t cpt;            // chunks per tap: Cin / 64
  int32_t full, rag_k8;   // whole chunks (C / 64), and the 8-column blocks after them
  int32_t rows_w;         // packed rows behind one wave's TO / 4 tile rows: TO / 4 * K / G
  int32_t grid8;          // launched workgroups / 8 (the tile count rounded up to a multiple of 8)
  int32_t ntiles;         // npb * nob
  // input geometry (an FC product is B = N images of 1 x 1 pixel)
  int32_t H, W, Cin, KH, KW, sh, sw, ph, pw;
  Div fd_nob, fd_howo, fd_wo, fd_cpt;
  uint32_t kw_mul;        // tap / KW == (tap * kw_mul) >> 16 for the taps (at most 32)
  uint32_t k_mul;         // r / K == (r * k_mul) >> 16 for the packed rows of a wave (at most 32)
  int32_t lg_g;           // log2 G
};

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Wait until at most N vector-memory operations of this wave are in flight
// (loads complete in issue order).
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt is 6 bits");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// Packed-weight loads into registers, issued as plain instructions that the
// compiler does not count (it would otherwise wait for the LDS DMAs issued
// after them); the kernel waits for them with wait_vm<> before any use.
__device__ __forceinline__ u32x4_t sdesc(const void* base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  const auto rfl = [](uint32_t x) { return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(x))); };
  return u32x4_t{rfl(static_cast<uint32_t>(a)), rfl(static_cast<uint32_t>(a >> 32) & 0xffffu), rfl(bytes),
                 static_cast<uint32_t>(kRsrcWord3)};
}
// (soff: a wave-uniform byte offset)
__device__ __forceinline__ u32x4_t load_x4(const u32x4_t d, uint32_t off, uint32_t soff) {
  u32x4_t v;
  asm volatile("buffer_load_dwordx4 %0, %1, %2, %3 offen" : "=v"(v) : "v"(off), "s"(d), "s"(soff) : "memory");
  return v;
}
__device__ __forceinline__ u32x2_t load_x2(const u32x4_t d, uint32_t off, uint32_t soff) {
  u32x2_t v;
  asm volatile("buffer_load_dwordx2 %0, %1, %2, %3 offen" : "=v"(v) : "v"(off), "s"(d), "s"(soff) : "memory");
  return v;
}

// f(integral_constant<int, K>) for K in the sequence, in order.
template <int... K, typename F>
__device__ __forceinline__ void for_k(std::integer_sequence<int, K...>, F&& f) {
  (f(std::integral_constant<int, K>{}), ...);
}

// acc += A * B on the matrix cores, with the accumulator pinned to the
// accumulation registers (the builtin lets the register allocator move the
// 64 accumulators between register files every chunk).  Dependent uses of
// acc by vector instructions are separated from the last MFMA by
// mfma_drain().  (volatile: kept in program order with the other volatile
// statements.)
__device__ __forceinline__ void mfma_acc(f32x4_t& acc, const bf16x8_t a, const bf16x8_t b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// Longer than any dependency between a vector write of an accumulation
// register and an MFMA reading it, or an MFMA result and a vector read.
__device__ __forceinline__ void mfma_drain() { asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory"); }
// Pin acc's current value in the accumulation registers at this point of
// the volatile sequence (no code).
__device__ __forceinline__ void acc_fence(f32x4_t& acc) { asm volatile("" : "+a"(acc)); }

// Ring stage K's packed units are used only after this point (after the
// wait that covers their loads).
template <int K, bool FULL, int RW, int UPL>
__device__ __forceinline__ void fence_stage(u32x4_t (&pv)[RW][UPL], u32x2_t (&pi)[RW][UPL]) {
#pragma unroll
  for (int u = 0; u < UPL; ++u) {
    asm volatile("" : "+v"(pv[K][u]));
    if constexpr (!FULL) asm volatile("" : "+v"(pi[K][u]));
  }
}

// Byte offset of tile row o (< 128) in the weight tile, k-column 0.
__device__ __forceinline__ uint32_t trow(uint32_t o) { return ((o >> 4) << 11) | ((o & 15) << 4); }

// UPL: 8-channel packed units per lane per chunk.  FULL: K == G (every
// entry kept, indices ascending, so a unit is one tile row's 16 bytes).
// BIGG: G == 32 (a group spans two 16-row blocks).  MASK: some lanes have no
// unit (else the checks compile away).
//
// KS: teams of four waves in the workgroup.  With two, team h takes the h-th
// half of the chunks, each team in LDS buffers of its own, and the partial
// tiles are added at the end: where the grid leaves one workgroup per CU, a
// SIMD then holds two waves whose LDS latencies, waits and tile builds
// overlap (the chunk loop of a lone team is bound by them, not by memory:
// prefetching deeper did not change it).
template <typename YT, int UPL, bool FULL, bool BIGG, bool MASK, int KS, int TO>
__device__ __forceinline__ void tap_tile_body(const TParams& p, uint8_t* const lds0) {
  constexpr int NX = kNX;
  constexpr int RW = 2;              // packed-unit ring stages
  constexpr int OT = TO / 32;        // 16-output tiles per wave
  constexpr int RPW = TO / 4;        // weight-tile rows a wave builds
  constexpr int WB = wb_bytes(TO);   // one weight tile
  constexpr int PITCH = ep_pitch(TO);
  constexpr int NMF = 4 * OT;        // MFMAs of one k-step
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int w = wv & 3, team = KS > 1 ? wv >> 2 : 0;
  const int wp = w >> 1, wo = w & 1;  // pixel half, output half (TO / 2 outputs) of this wave
  uint8_t* const lds = lds0 + team * lds_bytes(TO);
  // this team's chunks: nch from chunk ch0 on (both teams run the same number
  // of steps; a chunk past the reduction is all zeros)
  const int nch = team_chunks(p.nch, KS), ch0 = team * nch;

  // ---- tile of this workgroup ---------------------------------------------
  // Dispatch places workgroup b on XCD b % 8; L numbers the workgroups of one
  // XCD consecutively, output block fastest, so the tiles that read the same
  // activations run behind one L2.  (The grid is rounded up to a multiple
  // of 8; the workgroups past the last tile leave at once.)
  const uint32_t bid = blockIdx.x;
  const uint32_t L = (bid & 7u) * static_cast<uint32_t>(p.grid8) + (bid >> 3);
  if (L >= static_cast<uint32_t>(p.ntiles)) return;
  uint32_t ob;
  const uint32_t pb = divmod(L, p.fd_nob, ob);

  // (The set-up below runs once per workgroup, before its first load, with two
  // waves on a SIMD: compiler-made divisions and a walk over the taps took
  // 5700 of the 12 000 cycles before the first MFMA of a 3x3 layer, 2800 of
  // 9600 of a 1x1 layer.)
  // ---- activation DMA ---------------------------------------------------------
  // DMA instruction i of wave w fills pixels (4 w + i) * 8 .. +7 of a buffer:
  // lane l writes the 16 bytes at (4 w + i) * 1024 + 16 l, i.e. pixel
  // q = (4 w + i) * 8 + l / 8, column l % 8, which holds channel block
  // (l % 8) ^ sw(q).  xbase: byte offset of that block of the input pixel
  // under tap (0, 0) (negative in the padding); xinv bit t: tap t of the
  // pixel falls into the padding, or the pixel is past N.
  const __amdgpu_buffer_rsrc_t xr =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.X), (short)0, static_cast<int>(p.x_bytes), kRsrcWord3);
  int32_t xbase[4];
  uint32_t xinv[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int q = (4 * w + i) * 8 + (lane >> 3);
    const int px = static_cast<int>(pb) * kTP + q;
    const int k8 = (lane & 7) ^ ((q >> 1) & 7);
    xbase[i] = 0;
    xinv[i] = ~0u;
    if (px < p.N) {
      uint32_t rem, ow;
      const uint32_t img = divmod(static_cast<uint32_t>(px), p.fd_howo, rem);
      const uint32_t oh = divmod(rem, p.fd_wo, ow);
      const int ih0 = static_cast<int>(oh) * p.sh - p.ph, iw0 = static_cast<int>(ow) * p.sw - p.pw;
      xbase[i] = ((static_cast<int>(img) * p.H + ih0) * p.W + iw0) * p.Cin * 2 + k8 * 16;
      // columns kw of the filter inside the image: lo <= kw < hi
      const int lo = max(0, -iw0), hi = min(p.KW, p.W - iw0);
      const uint32_t row = hi > lo ? (hi < 32 ? (1u << hi) - 1u : ~0u) & (~0u << lo) : 0u;
      uint32_t ok = 0;
      for (int kh = 0; kh < p.KH; ++kh)
        ok |= static_cast<unsigned>(ih0 + kh) < static_cast<unsigned>(p.H) ? row << (kh * p.KW) : 0u;
      xinv[i] = ~ok;
    }
  }
  // Tap cursor of the next chunk to DMA: t = tap (row kh, column kw of the
  // filter), cb = channel block.  The lane's byte offsets under that tap (bit
  // 31 set where the tap falls into the padding) change with the tap only, the
  // channel block is the loads' uniform offset: they are kept (xv) where the
  // registers allow it (one packed unit per lane), else made per chunk.
  constexpr bool KEEP = UPL == 1;
  uint32_t cb0;
  int cur_t = static_cast<int>(divmod(static_cast<uint32_t>(ch0), p.fd_cpt, cb0)), cur_cb = static_cast<int>(cb0);
  int cur_kh = static_cast<int>(static_cast<uint32_t>(cur_t) * p.kw_mul >> 16), cur_kw = cur_t - cur_kh * p.KW;
  uint32_t xv[KEEP ? 4 : 1];
  const auto tap_off = [&](int i) {
    // (after the last of 32 taps cur_t is 32: only a dead chunk, every bit of
    // its xinv set, still loads)
    return static_cast<uint32_t>(xbase[i] + (cur_kh * p.W + cur_kw) * p.Cin * 2) |
           (((xinv[i] >> (cur_t & 31)) & 1u) << 31);
  };
  auto set_tap = [&] {
    if constexpr (KEEP) {
#pragma unroll
      for (int i = 0; i < 4; ++i) xv[i] = tap_off(i);
    }
  };
  set_tap();
  // From chunk `full` on the column blocks past C read zero, in X here and in
  // the packed rows in load_w, so that a neighbouring row's infinity cannot
  // meet a zero.  (TAIL: the chunk may be such a one; a dead chunk after them
  // leaves every offset out of range.)
  const int rag = p.full - ch0;  // the first chunk of this team that is not whole
  const auto live_k8 = [&](int ch) { return ch == rag ? p.rag_k8 : 0; };
  auto issue_x = [&](int ch, int buf, auto tail) {
    uint8_t* dst = lds + buf * kXB + w * 4096;
    if constexpr (decltype(tail)::value) {
      if (ch >= rag) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int q = (4 * w + i) * 8 + (lane >> 3);
          const bool live = ((lane & 7) ^ ((q >> 1) & 7)) < live_k8(ch);
          xinv[i] = live ? xinv[i] : ~0u;
          if constexpr (KEEP) xv[i] = live ? xv[i] : kOOB;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_void_t*)(dst + i * 1024), 16, KEEP ? xv[KEEP ? i : 0] : tap_off(i),
                                               cur_cb * (kCK * 2), 0, 0);
    if (++cur_cb == p.cpt) {
      cur_cb = 0;
      ++cur_t;
      if (++cur_kw == p.KW) {
        cur_kw = 0;
        ++cur_kh;
      }
      set_tap();
    }
  };

  // ---- packed weights ---------------------------------------------------------
  // Wave w expands tile rows [RPW w, RPW w + RPW): RPW / G groups, rows_w
  // packed rows.  Unit u of a lane is packed row r = (lane + 64 u) / 8 of them,
  // channels 8 c8 .. +7 of the chunk, c8 = (lane + 64 u) % 8.
  const u32x4_t vd = sdesc(p.vals, p.v_bytes), id = sdesc(p.idx, p.i_bytes);
  // The lanes of one packed row write neighbouring column blocks whose
  // 16-byte row segments all start on the same bank, so at step e lane l
  // writes element e ^ m, m = 2 (l % 4), of its unit: one instruction's
  // two-byte stores spread over four times as many banks (the halves of a
  // bank word need no spreading).  A unit's values and indices are permuted
  // once (permute_unit) so that step e reads them at fixed positions.
  const uint32_t m = 2u * static_cast<uint32_t>(lane & 3);
  uint32_t voff[UPL], ioff[UPL], ubase[UPL];
  bool uok[UPL];
#pragma unroll
  for (int u = 0; u < UPL; ++u) {
    const int v = lane + 64 * u;
    const int r = v >> 3, c8 = v & 7;
    uok[u] = !MASK || r < p.rows_w;
    const uint32_t prow = (ob * static_cast<uint32_t>(TO >> p.lg_g) + static_cast<uint32_t>(w * (RPW >> p.lg_g))) *
                              static_cast<uint32_t>(p.K) +
                          static_cast<uint32_t>(r);
    voff[u] = uok[u] ? (prow * static_cast<uint32_t>(p.C) + static_cast<uint32_t>(c8 * 8)) * 2u : kOOB;
    ioff[u] = uok[u] ? prow * static_cast<uint32_t>(p.C) + static_cast<uint32_t>(c8 * 8) : kOOB;
    // first tile row of the unit's group
    const int o0 = RPW * w + (FULL ? r : static_cast<int>(static_cast<uint32_t>(r) * p.k_mul >> 16) << p.lg_g);
    // (non-FULL: bits 1..3 carry 2 m, the byte offset of element m)
    ubase[u] = trow(static_cast<uint32_t>(uok[u] ? o0 : 0)) +
               static_cast<uint32_t>((c8 >> 2) * 1024 + (c8 & 3) * 256) + (FULL ? 0u : 2u * m);
  }
  // Register ring of RW stages: stage k holds the packed units of the
  // chunks j with j % RW == k (the index is always a compile-time constant).
  u32x4_t pv[RW][UPL];
  u32x2_t pi[RW][UPL];
  auto load_w = [&](int ch, auto kc, auto tail) {
    constexpr int k = decltype(kc)::value;
    if constexpr (decltype(tail)::value) {
      if (ch >= rag && (lane & 7) >= live_k8(ch)) {  // (c8 of every unit of a lane is lane % 8)
#pragma unroll
        for (int u = 0; u < UPL; ++u) voff[u] = ioff[u] = kOOB;
      }
    }
    const uint32_t at = static_cast<uint32_t>(decltype(tail)::value ? load_chunk(ch0 + ch, p.nch) : ch0 + ch);
#pragma unroll
    for (int u = 0; u < UPL; ++u) {
      pv[k][u] = load_x4(vd, voff[u], at * (kCK * 2));
      if constexpr (!FULL) pi[k][u] = load_x2(id, ioff[u], at * kCK);
    }
  };
  auto w_fence = [&](auto kc) { fence_stage<decltype(kc)::value, FULL>(pv, pi); };
  auto permute_unit = [&](auto kc, int u) {  // element e of the unit moves to position e ^ m
    constexpr int k = decltype(kc)::value;
    if constexpr (!FULL) {
      u32x4_t d = pv[k][u];
      u32x2_t x = pi[k][u];
      if (m & 4u) {
        d = u32x4_t{d[2], d[3], d[0], d[1]};
        x = u32x2_t{x[1], x[0]};
      }
      if (m & 2u) d = u32x4_t{d[1], d[0], d[3], d[2]};
      pv[k][u] = d;
      pi[k][u] = u32x2_t{__builtin_amdgcn_alignbit(x[0], x[0], 8u * (m & 2u)),
                         __builtin_amdgcn_alignbit(x[1], x[1], 8u * (m & 2u))};
    }
  };
  // tile offset of row rr of a group, relative to its first row
  auto grow = [](uint32_t rr) { return BIGG ? trow(rr) : rr << 4; };
  // Building a tile: wave w zeroes its RPW rows (RPW / 16 blocks of 16 rows,
  // both k-steps: RPW * 128 bytes at w * RPW * 128), then
  // writes its kept weights; LDS operations of one wave complete in order.
  auto zero_piece = [&](uint8_t* tb, int i) {
    *reinterpret_cast<u32x4_t*>(tb + w * (RPW * 128) + i * 1024 + lane * 16) = u32x4_t{0u, 0u, 0u, 0u};
  };
  auto scatter_e = [&](uint8_t* tb, auto kc, int u, int e) {  // step e of unit u (element e ^ m)
    constexpr int k = decltype(kc)::value;
    if (!uok[u]) return;
    if constexpr (FULL) {
      if (e == 0) *reinterpret_cast<u32x4_t*>(tb + ubase[u]) = pv[k][u];
    } else {
      // row within the group (masked to the group's span: a bad index byte
      // cannot address past the tile)
      // (bits 1..3 of ubase hold 2 m and rows move bits 4 and up: element e
      // ^ m's byte offset is 2 e flipped into them, before or after the row is
      // added.  Before makes it a loop constant per e, one instruction less,
      // where the registers hold eight of them: one unit per lane.)
      const uint32_t rr = __builtin_amdgcn_ubfe(pi[k][u][e >> 2], 8 * (e & 3), BIGG ? 5 : 4);
      const uint32_t at = UPL == 1 ? (ubase[u] ^ (2u * static_cast<uint32_t>(e))) + grow(rr)
                                   : (ubase[u] + grow(rr)) ^ (2u * static_cast<uint32_t>(e));
      *reinterpret_cast<uint16_t*>(tb + at) =
          static_cast<uint16_t>(pv[k][u][e >> 1] >> (16 * (e & 1)));
    }
  };

  // ---- MFMAs ------------------------------------------------------------------
  // acc[pt][ot]: 16 pixels (tile pt of the wave's 64) x 16 outputs (tile ot
  // of its TO / 2).  A lane holds outputs 4 (lane / 16) .. +3 of pixel
  // lane % 16.
  f32x4_t acc[4][OT];
#pragma unroll
  for (int pt = 0; pt < 4; ++pt)
#pragma unroll
    for (int ot = 0; ot < OT; ++ot) acc[pt][ot] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int pt = 0; pt < 4; ++pt)
#pragma unroll
    for (int ot = 0; ot < OT; ++ot) acc_fence(acc[pt][ot]);
  mfma_drain();  // the zero writes land before the first MFMA reads them
  // B fragment (activations): pixel lane % 16, channels 8 (4 s + lane / 16) ..
  const uint32_t xl = static_cast<uint32_t>(lane & 15), xk = static_cast<uint32_t>(lane >> 4);
  const uint32_t swz = (xl >> 1) & 7u;
  const uint32_t boff0 = xl * 128u + ((xk ^ swz) << 4), boff1 = xl * 128u + (((4u + xk) ^ swz) << 4);
  auto ld = [](const uint8_t* q) { return *reinterpret_cast<const bf16x8_t*>(q); };

  // ---- pipeline -----------------------------------------------------------------
  // A wave's vector-memory operations are issued in pairs W(m), X(m) (packed
  // units into ring stage m % 2, activations into buffer m % 3): m = 0, 1, 2
  // before the loop, then m = j + 3 in the second half of chunk j: chunk j has
  // released the buffer, and tile j+1, built in its first half, the stage.
  // Loads complete in issue order, so "W(j+1) has landed" is "at most X(j+1)
  // and the pairs issued after it are in flight".
  constexpr int kPair = (FULL ? 1 : 2) * UPL + 4;  // vector-memory operations of one pair
  static_assert(2 * kPair < 64, "vmcnt range");
  const auto wbuf = [&](int j) { return lds + NX * kXB + (j & 1) * WB; };
  bf16x8_t fa[OT], fb[4], ga[OT], gb[4];  // fragments of k-step 0, of k-step 1
  const auto read_fa = [&](int j, int q) { fa[q] = ld(wbuf(j) + wo * (OT * 2048) + lane * 16 + (2 * q) * 1024); };
  const auto read_fb = [&](int j, int q) { fb[q] = ld(lds + (j % NX) * kXB + wp * 8192 + q * 2048 + boff0); };
  for_k(std::make_integer_sequence<int, RW>{}, [&](auto kc) {
    if (decltype(kc)::value < nch) {
      load_w(decltype(kc)::value, kc, std::integral_constant<bool, true>{});
      issue_x(decltype(kc)::value, decltype(kc)::value, std::integral_constant<bool, true>{});
    }
  });
  if (nch > 1) wait_vm<kPair>(); else wait_vm<0>();  // W(0), X(0)
  w_fence(std::integral_constant<int, 0>{});
  for (int u = 0; u < UPL; ++u) permute_unit(std::integral_constant<int, 0>{}, u);
  if constexpr (!FULL)
    for (int i = 0; i < RPW / 4; ++i) zero_piece(wbuf(i / (RPW / 8)), i % (RPW / 8));  // both tiles
  for (int u = 0; u < UPL; ++u)
    for (int e = 0; e < 8; ++e) scatter_e(wbuf(0), std::integral_constant<int, 0>{}, u, e);
  if (nch > 2) {
    load_w(2, std::integral_constant<int, 0>{}, std::integral_constant<bool, true>{});
    issue_x(2, 2, std::integral_constant<bool, true>{});
  }
  lds_barrier();
#pragma unroll
  for (int q = 0; q < OT; ++q) read_fa(0, q);
#pragma unroll
  for (int q = 0; q < 4; ++q) read_fb(0, q);

  // Chunk j with j % 2 == k in buffer x, its k-step-0 fragments in registers.  The MFMAs
  // are issued one by one with the other work placed between them (a wave
  // issues in order):
  //   k-step 0: the k-step-1 fragments, then the kept weights of tile j+1 (8
  //     UPL two-byte stores) into rows zeroed a chunk ago;
  //   barrier: chunk j's fragments are in registers everywhere, tile j+1 and
  //     X(j+1) are complete;
  //   k-step 1: the k-step-0 fragments of chunk j+1, the zero fill of tile
  //     j+2 (in tile j's rows), the pair W(j+3), X(j+3).
  // So a fragment read always has half a chunk of MFMAs to land in: with the
  // barrier after the chunk, every chunk began with an exposed LDS round trip
  // (us, before / with it and fewer address instructions: 4096 x 2048 -> 2048
  // 47 / 43; 3000 x 3008 -> 3008 87 / 80; 300 x 4096 -> 4096 33.6 / 31.5).
  // ST: the steady state, where chunks j+1 .. j+3 exist and are whole.
  auto step = [&](int j, int x, auto kc, auto st) {
    constexpr int k1 = (decltype(kc)::value + 1) % RW;
    constexpr bool ST = decltype(st)::value;
    const bool next = ST || j + 1 < nch, next2 = ST || j + 2 < nch, issue = ST || j + NX < nch;
    const uint8_t* xb = lds + x * kXB + wp * 8192;
    const uint8_t* xn = lds + (x == NX - 1 ? 0 : x + 1) * kXB + wp * 8192;
    const uint8_t* wb = wbuf(j) + wo * (OT * 2048) + lane * 16;
    if (next) {
      if (next2) wait_vm<kPair + 4>(); else wait_vm<4>();  // W(j+1)
      w_fence(std::integral_constant<int, k1>{});
#pragma unroll
      for (int u = 0; u < UPL; ++u) permute_unit(std::integral_constant<int, k1>{}, u);
    }
#pragma unroll
    for (int i = 0; i < NMF; ++i) {
      mfma_acc(acc[i / OT][i % OT], fa[i % OT], fb[i / OT]);
      __builtin_amdgcn_sched_barrier(0);
      if (i < OT) ga[i] = ld(wb + (2 * i + 1) * 1024);
      if (i >= OT && i < OT + 4) gb[i - OT] = ld(xb + (i - OT) * 2048 + boff1);
      if (next) {
        // step q of the 8 UPL stores goes to slot q * NMF / (8 UPL)
#pragma unroll
        for (int q = 0; q < 8 * UPL; ++q)
          if ((q * NMF) / (8 * UPL) == i) scatter_e(wbuf(j + 1), std::integral_constant<int, k1>{}, q >> 3, q & 7);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (next) {
      if (next2) wait_vm<kPair>(); else wait_vm<0>();  // X(j+1)
      lds_barrier();
    }
#pragma unroll
    for (int i = 0; i < NMF; ++i) {
      mfma_acc(acc[i / OT][i % OT], ga[i % OT], gb[i / OT]);
      __builtin_amdgcn_sched_barrier(0);
      if (next) {
        if (i < OT) read_fa(j + 1, i);
        if (i < 4) fb[i] = ld(xn + i * 2048 + boff0);
      }
      if constexpr (!FULL) {
        if (i >= NMF / 2 && i < NMF / 2 + RPW / 8 && next2) zero_piece(wbuf(j), i - NMF / 2);
      }
      if (i == NMF - 4 && issue) load_w(j + NX, std::integral_constant<int, k1>{}, std::integral_constant<bool, !ST>{});
      if (i == NMF - 3 && issue) issue_x(j + NX, x, std::integral_constant<bool, !ST>{});
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // two chunks per iteration of the steady state, so every ring stage is a
  // constant; the tail (up to six chunks: the last two may not be whole)
  // starts again at stage 0.  (A loop, not six copies: straight-line code is
  // fetched cold by every workgroup.)
  int j = 0, x = 0;
  const auto advance = [&] { x = x == NX - 1 ? 0 : x + 1; };
  const int whole = min(nch, rag);
#pragma unroll 1
  for (; j + NX + 1 < whole; j += RW)
    for_k(std::make_integer_sequence<int, RW>{}, [&](auto kc) {
      step(j + decltype(kc)::value, x, kc, std::integral_constant<bool, true>{});
      advance();
    });
#pragma unroll 1
  for (; j < nch; j += RW)
    for_k(std::make_integer_sequence<int, RW>{}, [&](auto kc) {
      constexpr int q = decltype(kc)::value;
      if (q == 0 || j + q < nch) step(j + q, x, kc, std::integral_constant<bool, false>{});
      advance();
    });
  lds_barrier();  // every wave has its last fragments: the operand buffers are free

  // ---- fused epilogue -----------------------------------------------------------
  // A wave parks its 64 / KS pixels x TO/2 outputs (fp32) in its own LDS region
  // (pitch TO/2 * 4 + 16 bytes: conflict-free both ways) and reads them back
  // by pixel rows: a lane then owns 8 consecutive outputs of one pixel (LPR
  // lanes cover the wave's TO/2), applies scale / bias / residual / ReLU in
  // fp32, rounds once and stores 16 (bf16) or 32 bytes.  With two teams, wave w of
  // team h finishes pixel tiles 2 h, 2 h + 1: it leaves its partial sums of
  // the other two tiles to wave w of the other team.
  constexpr int LPR = TO / 16;   // lanes per pixel row
  constexpr int RPP = 64 / LPR;  // rows per pass
  constexpr int NPT = 4 / KS;    // pixel tiles this wave finishes
  constexpr int NPS = LPR / KS;  // its passes
  mfma_drain();  // the last MFMAs have written acc
#pragma unroll
  for (int pt = 0; pt < 4; ++pt)
#pragma unroll
    for (int ot = 0; ot < OT; ++ot) acc_fence(acc[pt][ot]);
  constexpr uint32_t ysz = sizeof(YT);
  uint8_t* stg = lds0 + wv * (16 * NPT) * PITCH;
  const __amdgpu_buffer_rsrc_t yr =
      __builtin_amdgcn_make_buffer_rsrc(p.Y, (short)0, static_cast<int>(p.y_bytes), kRsrcWord3);
  const __amdgpu_buffer_rsrc_t rsr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(p.residual), (short)0, p.residual ? static_cast<int>(p.y_bytes) : 0, kRsrcWord3);
  const int c8 = lane % LPR;  // 8-output block of the wave's TO/2
  const uint32_t o = ob * TO + static_cast<uint32_t>(wo * (TO / 2) + 8 * c8);
  const bool o_ok = o < static_cast<uint32_t>(p.O);  // (O % 8 == 0: all of the lane's outputs or none)
  const auto row_off = [&](int rr) {  // Y / residual byte offset of the lane's row rr
    const uint32_t px = pb * kTP + static_cast<uint32_t>(wp * 64 + 16 * NPT * team + RPP * rr + lane / LPR);
    return px < static_cast<uint32_t>(p.N) && o_ok ? (px * static_cast<uint32_t>(p.O) + o) * ysz : kOOB;
  };
  f32x4_t sc0{1.f, 1.f, 1.f, 1.f}, sc1{1.f, 1.f, 1.f, 1.f}, bi0{0.f, 0.f, 0.f, 0.f}, bi1{0.f, 0.f, 0.f, 0.f};
  if (p.scale && o_ok) {
    sc0 = *reinterpret_cast<const f32x4_t*>(p.scale + o);
    sc1 = *reinterpret_cast<const f32x4_t*>(p.scale + o + 4);
  }
  if (p.bias && o_ok) {
    bi0 = *reinterpret_cast<const f32x4_t*>(p.bias + o);
    bi1 = *reinterpret_cast<const f32x4_t*>(p.bias + o + 4);
  }
  // bf16 residual: all rows' 16-byte pieces are requested before the
  // accumulators are parked (one load latency, not one per row)
  u32x4_t rres[NPS];
  if constexpr (ysz == 2) {
    if (p.residual) {
#pragma unroll
      for (int rr = 0; rr < NPS; ++rr)
        rres[rr] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rsr, row_off(rr), 0, 0));
    }
  }
  const auto slot = [&](uint8_t* region, int q, int ot) {  // block (q, ot) of a region
    return reinterpret_cast<f32x4_t*>(region + (q * 16 + (lane & 15)) * PITCH + (ot * 16 + 4 * (lane >> 4)) * 4);
  };
  if constexpr (KS == 1) {
#pragma unroll
    for (int pt = 0; pt < 4; ++pt)
#pragma unroll
      for (int ot = 0; ot < OT; ++ot) *slot(stg, pt, ot) = acc[pt][ot];
  } else {
    // the partner finds this wave's partial sums in its own region and adds
    // its accumulators to them in place
    uint8_t* const other = lds0 + (wv ^ 4) * (16 * NPT) * PITCH;
    for_k(std::make_integer_sequence<int, KS>{}, [&](auto hc) {
      constexpr int H = decltype(hc)::value;
      if (team == H) {
#pragma unroll
        for (int q = 0; q < NPT; ++q)
#pragma unroll
          for (int ot = 0; ot < OT; ++ot) *slot(other, q, ot) = acc[NPT * (1 - H) + q][ot];
      }
    });
    lds_barrier();
    for_k(std::make_integer_sequence<int, KS>{}, [&](auto hc) {
      constexpr int H = decltype(hc)::value;
      if (team == H) {
#pragma unroll
        for (int q = 0; q < NPT; ++q)
#pragma unroll
          for (int ot = 0; ot < OT; ++ot) *slot(stg, q, ot) += acc[NPT * H + q][ot];
      }
    });
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // this wave's staging writes have landed
  // (A lane reads back what it owns: no other lane waits for it.  One look at
  // all sums first: the loop, one row's LDS latency after the other, takes 0.9
  // us of 15 where nothing is to be done.)
  uint32_t top = 0;
  if (p.kept_only) {
#pragma unroll
    for (int rr = 0; rr < NPS; ++rr) {
      const u32x4_t* const src = reinterpret_cast<const u32x4_t*>(stg + (RPP * rr + lane / LPR) * PITCH + c8 * 32);
#pragma unroll
      for (int e = 0; e < 4; ++e) top = max(top, max(src[0][e] & 0x7fffffffu, src[1][e] & 0x7fffffffu));
    }
  }
  if (__any(top >= 0x7f800000u)) {
#pragma unroll 1
    for (int rr = 0; rr < NPS; ++rr) {
      f32x4_t* const src = reinterpret_cast<f32x4_t*>(stg + (RPP * rr + lane / LPR) * PITCH + c8 * 32);
      const f32x4_t h0 = src[0], h1 = src[1];
      float y[8] = {h0[0], h0[1], h0[2], h0[3], h1[0], h1[1], h1[2], h1[3]};
      const uint32_t px = pb * kTP + static_cast<uint32_t>(wp * 64 + 16 * NPT * team + RPP * rr + lane / LPR);
      keep_kept<true>(y, p, p.K, static_cast<int32_t>(px), static_cast<int32_t>(o),
                      px < static_cast<uint32_t>(p.N) && o_ok);
      src[0] = f32x4_t{y[0], y[1], y[2], y[3]};
      src[1] = f32x4_t{y[4], y[5], y[6], y[7]};
    }
  }
#pragma unroll
  for (int rr = 0; rr < NPS; ++rr) {
    const int row = RPP * rr + lane / LPR;
    const uint8_t* src = stg + row * PITCH + c8 * 32;
    f32x4_t y0 = *reinterpret_cast<const f32x4_t*>(src);
    f32x4_t y1 = *reinterpret_cast<const f32x4_t*>(src + 16);
    const uint32_t off = row_off(rr);
    y0 = y0 * sc0 + bi0;
    y1 = y1 * sc1 + bi1;
    if (p.residual) {
      if constexpr (ysz == 2) {
        const u32x4_t r = rres[rr];
        y0[0] += __uint_as_float(r[0] << 16);
        y0[1] += __uint_as_float(r[0] & 0xffff0000u);
        y0[2] += __uint_as_float(r[1] << 16);
        y0[3] += __uint_as_float(r[1] & 0xffff0000u);
        y1[0] += __uint_as_float(r[2] << 16);
        y1[1] += __uint_as_float(r[2] & 0xffff0000u);
        y1[2] += __uint_as_float(r[3] << 16);
        y1[3] += __uint_as_float(r[3] & 0xffff0000u);
      } else {
        y0 += __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rsr, off, 0, 0));
        y1 += __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rsr, off + 16, 0, 0));
      }
    }
    if (p.relu) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        y0[e] = y0[e] > 0.0f ? y0[e] : (y0[e] != y0[e] ? y0[e] : 0.0f);
        y1[e] = y1[e] > 0.0f ? y1[e] : (y1[e] != y1[e] ? y1[e] : 0.0f);
      }
    }
    if constexpr (ysz == 2) {
      // v_cvt_pk_bf16_f32: round to nearest even
      const u32x4_t pk = {__builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{y0[0], y0[1]}), bf16x2_t)),
                          __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{y0[2], y0[3]}), bf16x2_t)),
                          __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{y1[0], y1[1]}), bf16x2_t)),
                          __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{y1[2], y1[3]}), bf16x2_t))};
      __builtin_amdgcn_raw_buffer_store_b128(
          __builtin_bit_cast(decltype(__builtin_amdgcn_raw_buffer_load_b128(yr, 0, 0, 0)), pk), yr, off, 0, 0);
    } else {
      __builtin_amdgcn_raw_buffer_store_b128(
          __builtin_bit_cast(decltype(__builtin_amdgcn_raw_buffer_load_b128(yr, 0, 0, 0)), y0), yr, off, 0, 0);
      __builtin_amdgcn_raw_buffer_store_b128(
          __builtin_bit_cast(decltype(__builtin_amdgcn_raw_buffer_load_b128(yr, 0, 0, 0)), y1), yr, off + 16, 0, 0);
    }
  }
}

template <typename YT, int UPL, bool FULL, bool BIGG, bool MASK, int KS, int TO>
__global__ __launch_bounds__(kThreads * KS) __attribute__((amdgpu_waves_per_eu(2, 2)))
void tap_tile_kernel(TParams p) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  tap_tile_body<YT, UPL, FULL, BIGG, MASK, KS, TO>(p, lds);
}

template <typename YT, int UPL, bool FULL, bool BIGG, bool MASK, int KS, int TO>
hipError_t launch_tn(const TParams& p, hipStream_t s) {
  static std::atomic<int8_t> lds_set[kMaxDevices];
  const hipError_t attr =
      set_lds_limit_once(lds_set, reinterpret_cast<const void*>(&tap_tile_kernel<YT, UPL, FULL, BIGG, MASK, KS, TO>),
                         KS * lds_bytes(TO));
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((tap_tile_kernel<YT, UPL, FULL, BIGG, MASK, KS, TO>), dim3(8u * static_cast<uint32_t>(p.grid8)),
                     dim3(kThreads * KS), KS * lds_bytes(TO), s, p);
  return hipGetLastError();
}

// Two one-team workgroups per CU once the grid covers every CU twice; below
// that one workgroup of two teams, if each has a few chunks (us, one team
// with a fourth activation buffer / two teams: 12544 x 1024 -> 256 18.5 /
// 16.3; 3136 x 4608 -> 512 44 / 36; 1537 x 2048 -> 1000 25.4 / 21.0; 300 x
// 4096 -> 4096 43.4 / 33.6).
template <typename YT, int UPL, bool FULL, bool BIGG, bool MASK, int TO>
hipError_t launch_tu(const TParams& p, hipStream_t s) {
  return static_cast<uint32_t>(p.ntiles) >= kPairGrid || p.nch < kPairChunks
             ? launch_tn<YT, UPL, FULL, BIGG, MASK, 1, TO>(p, s)
             : launch_tn<YT, UPL, FULL, BIGG, MASK, 2, TO>(p, s);
}

template <typename YT, bool BIGG, int TO>
hipError_t launch_tg(const TParams& p, hipStream_t s) {
  // units per wave: 8 rows_w; per lane: rows_w / 8, rounded up (rows_w <= 16:
  // at most half of a group kept)
  if (p.rows_w < 8) return launch_tu<YT, 1, false, BIGG, true, TO>(p, s);
  if (p.rows_w == 8) return launch_tu<YT, 1, false, BIGG, false, TO>(p, s);
  if constexpr (TO == 128) {
    if (p.rows_w < 16) return launch_tu<YT, 2, false, BIGG, true, TO>(p, s);
    return launch_tu<YT, 2, false, BIGG, false, TO>(p, s);
  }
  return hipErrorInvalidConfiguration;  // (TO = 64: rows_w <= 8)
}

template <typename YT>
hipError_t launch_ty(const TParams& p, hipStream_t s, int to) {
  if (to == 64) {
    if (p.K == p.G) return launch_tu<YT, 2, true, false, false, 64>(p, s);
    return launch_tg<YT, false, 64>(p, s);
  }
  if (p.K == p.G) return launch_tu<YT, 4, true, false, false, 128>(p, s);
  return p.G == 32 ? launch_tg<YT, true, 128>(p, s) : launch_tg<YT, false, 128>(p, s);
}

}  // namespace

bool tap_tile_supports(const ProductArgs& a) {
  if (a.x_t != DType::BF16 || a.val_t != DType::BF16) return false;
  if (a.G < 1 || a.G > 32 || 32 % a.G != 0 || a.K < 1 || a.K > a.G) return false;
  // at most half of each group kept, or all of it (dense control): above
  // that the packed units no longer fit the registers beside the rings
  if (2 * a.K > a.G && a.K != a.G) return false;
  // a lane of the epilogue holds 8 outputs; G = 32 takes whole tiles of 128
  // outputs only (a group must fit the rows one wave builds)
  if (a.N < 1 || a.O % 8 != 0 || (a.O % 128 != 0 && a.G > 16)) return false;
  // chunks of 64 columns under one tap; the last chunk of a single tap's
  // reduction may be short (in blocks of 8 columns)
  const int64_t cin = a.conv ? a.geom.Cin : a.C;
  if (cin % kCK != 0 && (cin != a.C || cin % 8 != 0)) return false;
  if (!a.ragged && (cin % kCK != 0 || a.O % 64 != 0)) return false;
  if (a.conv && a.geom.KH * a.geom.KW > kMaxTaps) return false;
  const auto al = [](const void* q, uintptr_t m) { return (reinterpret_cast<uintptr_t>(q) & (m - 1)) == 0; };
  if (!al(a.X, 16) || !al(a.vals, 16) || !al(a.idx, 8) || !al(a.Y, 16)) return false;
  if ((a.scale && !al(a.scale, 16)) || (a.bias && !al(a.bias, 16)) || (a.residual && !al(a.residual, 16)))
    return false;
  // every buffer offset is 32-bit and stays below the out-of-range marker
  const int64_t lim = static_cast<int64_t>(kOOB);
  const int64_t x_elems = a.conv ? a.B * a.geom.H * a.geom.W * a.geom.Cin : a.N * a.C;
  const int64_t packed = (a.O / a.G) * a.K * a.C;
  if (x_elems * 2 >= lim || packed * 2 >= lim || a.N * a.O * (a.y_t == DType::F32 ? 4 : 2) >= lim) return false;
  return true;
}

hipError_t launch_tap_tile(const ProductArgs& a, hipStream_t s) {
  if (!tap_tile_supports(a)) return hipErrorInvalidConfiguration;
  TParams p{};
  p.X = static_cast<const uint16_t*>(a.X);
  p.vals = static_cast<const uint16_t*>(a.vals);
  p.idx = a.idx;
  p.scale = a.scale;
  p.bias = a.bias;
  p.residual = a.residual;
  p.Y = a.Y;
  const int64_t ysz = a.y_t == DType::F32 ? 4 : 2;
  const int64_t packed = (a.O / a.G) * a.K * a.C;
  if (a.conv) {
    const ConvGeom& g = a.geom;
    p.x_bytes = static_cast<uint32_t>(a.B * g.H * g.W * g.Cin * 2);
    p.H = g.H;
    p.W = g.W;
    p.Cin = g.Cin;
    p.KH = g.KH;
    p.KW = g.KW;
    p.sh = g.sh;
    p.sw = g.sw;
    p.ph = g.ph;
    p.pw = g.pw;
    p.fd_howo = make_div(static_cast<int64_t>(g.Ho) * g.Wo);
    p.fd_wo = make_div(g.Wo);
  } else {  // N images of one pixel
    p.x_bytes = static_cast<uint32_t>(a.N * a.C * 2);
    p.H = p.W = 1;
    p.Cin = static_cast<int32_t>(a.C);
    p.KH = p.KW = 1;
    p.sh = p.sw = 1;
    p.ph = p.pw = 0;
    p.fd_howo = p.fd_wo = make_div(1);
  }
  p.kw_mul = (1u << 16) / static_cast<uint32_t>(p.KW) + 1;
  p.k_mul = (1u << 16) / static_cast<uint32_t>(a.K) + 1;
  while ((1 << p.lg_g) < a.G) ++p.lg_g;
  p.v_bytes = static_cast<uint32_t>(packed * 2);
  p.i_bytes = static_cast<uint32_t>(packed);
  p.y_bytes = static_cast<uint32_t>(a.N * a.O * ysz);
  p.N = static_cast<int32_t>(a.N);
  p.C = static_cast<int32_t>(a.C);
  p.O = static_cast<int32_t>(a.O);
  p.G = a.G;
  p.K = a.K;
  p.relu = a.relu;
  p.kept_only = a.kept_only;
  p.npb = static_cast<int32_t>((a.N + kTP - 1) / kTP);
  // 128-output tiles, unless they would leave more than half of the CUs idle
  // or one of them would be more than half empty (us, 128 / 64 outputs:
  // 12544 x 1024 -> 256, 196 tiles, 16.3 / 19.9; 12544 x 816 -> 136, 196
  // tiles, 15.6 / 17.4; 1537 x 2048 -> 1000, 104 tiles, 23.2 / 20.0; 12544 x
  // 576 -> 96, 98 tiles, 12.7 / 10.6; 50176 x 288 -> 48 14.5 / 12.3).
  // G = 32 has no 64-output form.
  const int64_t grid128 = static_cast<int64_t>(p.npb) * ((a.O + 127) / 128);
  const int to = a.G > 16 || (grid128 >= kSmallGrid && a.O > 64) ? 128 : 64;
  p.nob = static_cast<int32_t>((a.O + to - 1) / to);
  p.nch = static_cast<int32_t>((a.C + kCK - 1) / kCK);
  p.cpt = (p.Cin + kCK - 1) / kCK;
  p.fd_nob = make_div(p.nob);
  p.fd_cpt = make_div(p.cpt);
  p.full = static_cast<int32_t>(a.C / kCK);
  p.rag_k8 = static_cast<int32_t>(a.C % kCK / 8);
  p.rows_w = to / 4 * a.K / a.G;
  const int64_t grid = static_cast<int64_t>(p.npb) * p.nob;
  if (grid > 0x7fffffff) return hipErrorInvalidConfiguration;
  p.ntiles = static_cast<int32_t>(grid);
  p.grid8 = static_cast<int32_t>((grid + 7) / 8);
  return a.y_t == DType::BF16 ? launch_ty<bf16_t>(p, s, to) : launch_ty<float>(p, s, to);
}

}  // namespace cci

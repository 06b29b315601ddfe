// bf16 MFMA main loop of the linear predictors (Sect. 3.2 of the AQUA-KV paper) for tiles of 32, 64, 96, 128, 192 or 320 token
// rows x 128 outputs (one kv head): the shapes a launch picks from so that its tiles fill the CUs evenly.
//
// Same instruction (v_mfma_f32_32x32x16_bf16), operand orientation, swizzled LDS layout, direct-to-LDS loads and K order
// per output as gemm_core.h, hence the same bits.  One workgroup per CU.
//   * 32 rows: four waves split the 128 columns; 64 rows: eight, 96 rows: twelve (three per SIMD), each holding 32 of the rows.  Such a tile is bound by the stream of
//     operands from L2, (rows + 128) x 128 bytes per k-tile of 64, most of it W: a deep ring of k-tiles in LDS keeps it
//     coming, and a wave reads the fragments of a whole k-tile ahead (its steps of 16 k are one or two MFMAs long).
//     Measured with 32 rows: 0.18 us per k-tile = 57 bytes per cycle into a CU, of 64; a 256-row tile takes 0.6 to 0.9.
//     The next loads are issued behind the first MFMA of a k-tile, which covers them: ahead of it, where the compiler put them while
//     that was left to it, with two additions per fragment address, one tensor took 2 to 5 % longer (128 rows, uniform backbone, keys 7.34 -> 6.98 us).
//   * From 128 rows on: eight waves (two per SIMD) as 2 x 4, wave (wm, wn) holds columns 32 wn ... and every second block
//     of 32 rows: (MI + 1) / MI operand reads per MFMA, MI = rows / 64.  192 rows: twelve waves as 3 x 4, MI = 2.
#pragma once
#include "gemm_core.h"

#include <type_traits>

namespace aquakv {

template <int MB> struct TileShape;                   // MB = 32-row blocks of the tile
template <> struct TileShape<1> { static constexpr int kStages = 7; };       // x 20 KiB
template <> struct TileShape<2> { static constexpr int kStages = 6; };       // x 24 KiB: 0.31 us per k-tile; with four waves and 3 stages 0.385
template <> struct TileShape<3> { static constexpr int kStages = 5; };       // x 28 KiB
template <> struct TileShape<4> { static constexpr int kStages = 4; };       // x 32 KiB
template <> struct TileShape<6> { static constexpr int kStages = 3; };       // x 40 KiB
template <> struct TileShape<10> { static constexpr int kStages = 2; };      // x 56 KiB
template <int MB> struct Tile : TileShape<MB> {
  static constexpr int kRows = 32 * MB;
  static constexpr int WM = MB == 1 ? 1 : MB % 3 == 0 ? 3 : 2, WN = 4;
  static constexpr int kWaves = WM * WN, kThreads = kWaves * 64;
  static constexpr int MI = MB / WM;                  // 32-row blocks per wave
  static constexpr int kAhead = MB < 4 ? 4 : 1;       // fragments are read this many steps of 16 k ahead
  static constexpr int kATile = kRows * kRowBytes;
  static constexpr int kStage = kATile + 128 * kRowBytes;
  static constexpr int kLdsBytes = TileShape<MB>::kStages * kStage;
  // first row of block i of the waves with this wm
  static constexpr int block_row(int i, int wm) { return (i * WM + wm) * 32; }
};

// s_waitcnt vmcnt(n) lgkmcnt(0), n < 64
template <int N> __device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14)); }

// acc[i]: the 32 x 32 block at rows block_row(i, wm), columns 32 wn of the tile, wm = wave / 4, wn = wave % 4 (layout inside
// the block as in gemm_core.h).  x0 / x1 point at the tile's first row; `last`: index of its last valid row (rows behind it
// are read as that row).  W points at the tile's first output row, rows ldw apart.  start() fills acc with the sums to start from
// once the first k-tile has landed, and with it every load issued before.  Requires K = d0 + d1 a multiple of 128, d0 of 64.
// Ends with every LDS read of the calling wave returned; the caller puts a barrier before it reuses the LDS.
// The counts of loads in flight assume that nothing but this loop issues global loads while it runs.
template <int MB> struct TileLoop {
  using S = Tile<MB>;
  template <typename Start>
  static __device__ __forceinline__ void run(unsigned char* lds_base, const bf16_t* __restrict__ x0, int d0,
                                             const bf16_t* __restrict__ x1, int d1, const bf16_t* __restrict__ W, int ldw,
                                             int last, f32x16 (&acc)[S::MI], Start&& start);
};
template <int MB>
template <typename Start>
__device__ __forceinline__ void TileLoop<MB>::run(unsigned char* lds_base, const bf16_t* __restrict__ x0, int d0,
                                                  const bf16_t* __restrict__ x1, int d1, const bf16_t* __restrict__ W,
                                                  int ldw, int last, f32x16 (&acc)[S::MI], Start&& start) {
  constexpr int kRowsPerPiece = S::kThreads / 8;      // tile rows one load instruction of the workgroup fills
  constexpr int kPieceBytes = S::kThreads * 16;
  constexpr int kA = S::kRows / kRowsPerPiece, kB = (128 + kRowsPerPiece - 1) / kRowsPerPiece, kPieces = kA + kB;
  constexpr int kPart = 128 % kRowsPerPiece / 8;      // not 0: the last piece of W is a load of the first kPart waves only
  constexpr int kStages = S::kStages, kAhead = S::kAhead, MI = S::MI;
  constexpr int kBufs = kAhead == 1 ? 2 : kAhead;
  static_assert(kA * kRowsPerPiece == S::kRows && kPieces * (kStages - 1) < 64, "whole pieces; vmcnt range");
  typedef __attribute__((address_space(3))) unsigned char* lptr_t;
  typedef const __attribute__((address_space(1))) char* gptr_t;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / S::WN, wn = wave % S::WN;
  const int K = d0 + d1, nk = K / BK;
  const bool all_pieces = kPart == 0 || wave < kPart;

  const int ch16 = ((tid & 7) ^ ((tid >> 4) & 7)) * 16;
  int rowc[kA];
#pragma unroll
  for (int pc = 0; pc < kA; ++pc) {
    const int row = (tid >> 3) + pc * kRowsPerPiece;
    rowc[pc] = row < last ? row : last;
  }
  const uint32_t offW = (uint32_t)(tid >> 3) * (uint32_t)(ldw * 2) + ch16;
  const auto uniform_ptr = [](const char* p) {
    const uint64_t u = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
    return (gptr_t)(((uint64_t)hi << 32) | lo);
  };
  const lptr_t lds3 = (lptr_t)lds_base;
  auto load_piece = [&](int kt, int stage_off, int pc) {
    const int k0 = kt * BK;
    const lptr_t dst = lds3 + (stage_off + wave * 1024 + pc * kPieceBytes);     // x pieces fill the A tile, W pieces follow
    if (pc < kA) {
      const bool second = k0 >= d0;
      const int ld2 = __builtin_amdgcn_readfirstlane((second ? d1 : d0) * 2);
      const gptr_t xb = uniform_ptr(reinterpret_cast<const char*>(second ? x1 : x0) + (int64_t)(second ? k0 - d0 : k0) * 2);
      __builtin_amdgcn_global_load_lds(xb + ((uint32_t)__umul24(rowc[pc], ld2) + ch16), dst, 16, 0, 0);
    } else if (pc + 1 < kPieces || all_pieces) {
      const gptr_t wb = uniform_ptr(reinterpret_cast<const char*>(W) + ((int64_t)k0 * 2 + (int64_t)(pc - kA) * kRowsPerPiece * ldw * 2));
      __builtin_amdgcn_global_load_lds(wb + offW, dst, 16, 0, 0);
    }
  };

  struct Frag { bf16x8 v[MI + 1]; };
  const int frow = lane & 31, fk = lane >> 5;
  auto frag_off = [&](int ks, int pc) { return lds_off((pc < MI ? S::block_row(pc, wm) : wn * 32) + frow, ks * 2 + fk); };
  // Where waves read whole k-tiles ahead, a fragment's place in a stage is kept in a register (opaque: the compiler would share parts
  // of them and add twice for each read).
  int kept[kAhead == 4 ? 4 : 1][MI + 1];
  if constexpr (kAhead == 4) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int pc = 0; pc <= MI; ++pc) {
        kept[ks][pc] = frag_off(ks, pc);
        asm("" : "+v"(kept[ks][pc]));
      }
  }
  auto frag_piece = [&](int stage_off, int ks, Frag& f, int pc) {
    const int off = kAhead == 4 ? kept[kAhead == 4 ? ks : 0][pc] : frag_off(ks, pc);
    f.v[pc] = *reinterpret_cast<const bf16x8*>(lds_base + stage_off + off + (pc < MI ? 0 : S::kATile));
  };
  auto read_frag = [&](int stage_off, int ks, Frag& f) {
#pragma unroll
    for (int pc = 0; pc <= MI; ++pc) frag_piece(stage_off, ks, f, MI - pc);     // the W fragment first
  };
  // the MFMAs of one step; extra(m) is issued right behind MFMA m (sched_barrier keeps the order)
  auto mma = [&](const Frag& f, auto&& extra) {
#pragma unroll
    for (int m = 0; m < MI; ++m) {
      acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.v[m], f.v[MI], acc[m], 0, 0, 0);
      extra(m);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // at most N newer k-tiles may still be on their way (loads complete in issue order)
  auto wait_newer = [&](auto n) {
    constexpr int N = decltype(n)::value;
    if (all_pieces) wait_loads<N * kPieces % 64>();
    else wait_loads<N * (kPieces - 1) % 64>();
  };
  auto wait_tiles = [&](int tiles) {
    if (tiles <= 0) wait_newer(std::integral_constant<int, 0>{});
    else if (tiles == 1) wait_newer(std::integral_constant<int, 1>{});
    else if (kStages > 4 && tiles == 2) wait_newer(std::integral_constant<int, 2>{});
    else if (kStages > 5 && tiles == 3) wait_newer(std::integral_constant<int, 3>{});
    else if (kStages > 6 && tiles == 4) wait_newer(std::integral_constant<int, 4>{});
    else wait_newer(std::integral_constant<int, kStages - 2>{});
  };
  auto meet = [&] {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };

  const int first = nk < kStages ? nk : kStages;
#pragma unroll
  for (int t = 0; t < kStages; ++t)
    if (t < first) {
#pragma unroll
      for (int pc = 0; pc < kPieces; ++pc) load_piece(t, t * S::kStage, pc);
    }
  // tile 0 has landed: `first` - 1 newer ones may be out
  if (first == kStages) wait_newer(std::integral_constant<int, kStages - 1>{});
  else wait_tiles(first - 1);
  meet();
  Frag f[kBufs];
#pragma unroll
  for (int s = 0; s < kAhead; ++s) read_frag(0, s, f[s]);
  __builtin_amdgcn_sched_barrier(0);
  start();
  __builtin_amdgcn_sched_barrier(0);

  // k-tile t sits in the stage at `cur`, t + 1 in the one at `nxt`.  Before the step that first reads k-tile t + 1 it is
  // published; by then every wave's reads of tile t have returned, so its stage takes tile t + kStages.
  auto tile = [&](int t, int cur, int nxt, bool has_next, bool steady, bool do_load) {
    const auto publish = [&] {
      if (steady) wait_newer(std::integral_constant<int, kStages - 2>{});
      else wait_tiles(nk - 2 - t);
      meet();
    };
    if constexpr (kAhead == 4) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        if (s == 0 && has_next) publish();
        mma(f[s], [](int) {});
        if (s == 0 && do_load) {                      // behind the first MFMAs: their issue takes as long as one of those
#pragma unroll
          for (int pc = 0; pc < kPieces; ++pc) load_piece(t + kStages, cur, pc);
        }
        if (has_next) read_frag(nxt, s, f[s]);        // behind the MFMAs that used this buffer
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
#pragma unroll
      for (int s = 0; s < 3; ++s)
        mma(f[s & 1], [&](int m) {
          if (2 * m <= MI) frag_piece(cur, s + 1, f[(s + 1) & 1], MI - 2 * m);
          if (2 * m + 1 <= MI) frag_piece(cur, s + 1, f[(s + 1) & 1], MI - 2 * m - 1);
        });
      if (has_next) publish();
      constexpr int kItems = MI + 1 + kPieces, kPerMma = (kItems + MI - 1) / MI;
      mma(f[1], [&](int m) {
#pragma unroll
        for (int e = m * kPerMma; e < (m + 1) * kPerMma && e < kItems; ++e) {
          if (e <= MI) { if (has_next) frag_piece(nxt, 0, f[0], MI - e); }
          else if (do_load) load_piece(t + kStages, cur, e - MI - 1);
        }
      });
    }
  };
  const auto step = [](int s) { return s + S::kStage == S::kLdsBytes ? 0 : s + S::kStage; };
  int cur = 0, nxt = S::kStage, t = 0;
  for (; t + kStages < nk; ++t) {
    tile(t, cur, nxt, true, true, true);
    cur = nxt; nxt = step(nxt);
  }
  for (; t + 1 < nk; ++t) {
    tile(t, cur, nxt, true, false, false);
    cur = nxt; nxt = step(nxt);
  }
  tile(t, cur, nxt, false, false, false);
  settle_accumulators(acc);
}

}  // namespace aquakv

// bf16 MFMA main loop of the linear predictors (Sect. 3.2 of the AQUA-KV paper) for tiles of 32, 64, 96, 128, 192, 256 or 320 token
// rows x 128 outputs (one kv head): the shapes a launch picks from so that its tiles fill the CUs evenly.
//
// Operands, LDS layout, K order: gemm_core.h, hence the same bits on every tile.  One workgroup per CU.
//   * Waves 0 .. 3, one per SIMD, multiply: below 128 rows each takes all rows and a quarter of the columns, from 128 rows on half of either.
//     Waves 4 .. 7 load, so a multiplying wave issues MFMAs and fragment reads and nothing else: a load's address arithmetic and its
//     issue, 16 cycles each, are on another wave.  192 and 96 rows have four more waves, for the epilogue (three per SIMD, 168 registers).
//   * What counts for a wave that is alone with its SIMD's matrix core is that no MFMA waits: fragments are read three steps of 16 k ahead up
//     to 128 rows (one beyond, where a step has enough MFMAs to cover an LDS read's 60 cycles and the registers are taken), across
//     the barrier that publishes the next k-tile.
//   * LDS holds as many k-tiles as fit: from L2 a k-tile takes 1 to 2 us, several times its MFMAs on the small tiles.
// Cycles per k-tile of 64 at K = 1024, before (all waves load and multiply) and now, 32 cycles per MFMA of a SIMD being the floor:
//   32 rows 450 -> 331 (128; bound by (rows + 128) x 128 bytes from L2 at 60 bytes a cycle), 64 552 -> 400 (256), 96 707 -> 483 (384),
//   128 918 -> 608 (512), 192 1217 -> 844 (768), 256 1379 -> 1092 (1024), 320 1878 -> 1709 (1280).
// 256 rows and more run at 1.55 to 1.75 GHz on random operands (2.4 on zeros): there the power limit binds, not the issue.
#pragma once
#include "gemm_core.h"

#include <type_traits>

namespace aquakv {

template <int MB> struct TileShape;                   // MB = 32-row blocks of the tile
template <> struct TileShape<1> { static constexpr int kWaves = 8, kStages = 7; };       // x 20 KiB
template <> struct TileShape<2> { static constexpr int kWaves = 8, kStages = 6; };       // x 24 KiB
template <> struct TileShape<3> { static constexpr int kWaves = 12, kStages = 5; };      // x 28 KiB
template <> struct TileShape<4> { static constexpr int kWaves = 8, kStages = 4; };       // x 32 KiB
template <> struct TileShape<6> { static constexpr int kWaves = 12, kStages = 3; };      // x 40 KiB
template <> struct TileShape<8> { static constexpr int kWaves = 8, kStages = 3; };       // x 48 KiB
template <> struct TileShape<10> { static constexpr int kWaves = 8, kStages = 2; };      // x 56 KiB
template <int MB> struct Tile : TileShape<MB> {
  static constexpr int kRows = 32 * MB;
  static constexpr int kThreads = TileShape<MB>::kWaves * 64;
  static constexpr int WM = MB < 4 ? 1 : 2, WN = 4 / WM;      // the four multiplying waves
  static constexpr int MI = MB / WM, NJ = 4 / WN;     // their blocks of 32 x 32
  static constexpr int kAhead = MB < 6 ? 3 : 1;       // fragments are read this many steps of 16 k ahead
  static constexpr int kATile = kRows * kRowBytes;
  static constexpr int kStage = kATile + 128 * kRowBytes;
  static constexpr int kLdsBytes = TileShape<MB>::kStages * kStage;
  // first row of block i of the waves with this wm, first column of block j of those with this wn
  static constexpr int block_row(int i, int wm) { return (i * WM + wm) * 32; }
  static constexpr int block_col(int j, int wn) { return (wn * NJ + j) * 32; }
};
constexpr int kMulWaves = 4, kLoadWaves = 4;          // waves 0 .. 3 multiply, 4 .. 7 load, what is left waits for them

// s_waitcnt vmcnt(n) lgkmcnt(0), n < 64
template <int N> __device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14)); }

// acc[i][j] (waves 0 .. 3): the 32 x 32 block at rows block_row(i, wm), columns block_col(j, wn) of the tile, wm = wave / WN, wn = wave % WN
// (layout inside the block as in gemm_core.h).  x0 / x1 point at the tile's first row; `last`: index of its last valid row (rows behind it
// are read as that row).  W points at the tile's first output row, rows ldw apart.  start() fills acc with the sums to start from,
// in the multiplying waves; request() is called by every wave once, where it issues what the caller needs behind the loop.
// Requires K = d0 + d1 a multiple of 128, d0 of 64.
// Ends with every LDS read of the calling wave returned; the caller puts a barrier before it reuses the LDS.
template <int MB> struct TileLoop {
  using S = Tile<MB>;
  static constexpr int kStages = S::kStages, MI = S::MI, NJ = S::NJ;
  static constexpr int kPieces = (S::kRows + 128) / 8 / kLoadWaves;   // load instructions of a wave and k-tile, 8 rows each
  static_assert((S::kRows + 128) % (8 * kLoadWaves) == 0 && kPieces * (kStages - 1) < 64, "whole pieces; vmcnt range");

  static __device__ __forceinline__ void meet() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  }

  // A loading wave: its share of every k-tile, as many k-tiles ahead as there are stages.
  static __device__ __forceinline__ void load(unsigned char* lds_base, const bf16_t* __restrict__ x0, int d0, const bf16_t* __restrict__ x1,
                                              int d1, const bf16_t* __restrict__ W, int ldw, int last, int wave, int lane) {
    typedef __attribute__((address_space(3))) unsigned char* lptr_t;
    typedef const __attribute__((address_space(1))) char* gptr_t;
    const int nk = (d0 + d1) / BK;
    const auto uniform_ptr = [](const char* p) {
      const uint64_t u = reinterpret_cast<uint64_t>(p);
      const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u);
      const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
      return (gptr_t)(((uint64_t)hi << 32) | lo);
    };
    const lptr_t lds3 = (lptr_t)lds_base;
    // piece pc of this wave: rows 8 (pc kLoadWaves + wave) ... of the tile, the x rows first
    constexpr int kA = S::kRows / 8 / kLoadWaves;
    static_assert(S::kRows % (8 * kLoadWaves) == 0, "a piece is x or W for all waves");
    const int row0 = wave * 8 + (lane >> 3);
    const int ch16 = ((lane & 7) ^ ((row0 >> 1) & 7)) * 16;          // (32 rows further the chunk is the same)
    // Offsets from scalar bases: nothing but scalar instructions and the loads themselves per k-tile, so that the vector pipe is the
    // multiplying waves' own.  (Changed by an empty statement where they are used, they stay 32 bits wide.)
    uint32_t offx[kA], offW = (uint32_t)row0 * (uint32_t)(ldw * 2) + ch16;
    const auto rows_of = [&](int d) {
#pragma unroll
      for (int pc = 0; pc < kA; ++pc) {
        const int row = row0 + pc * 8 * kLoadWaves;
        offx[pc] = (uint32_t)__umul24(row < last ? row : last, d * 2) + ch16;
      }
    };
    rows_of(d0);
    gptr_t xb = uniform_ptr(reinterpret_cast<const char*>(x0)), wb = uniform_ptr(reinterpret_cast<const char*>(W));
    int k0 = 0;                                        // of the next k-tile
    const int64_t w_step = (int64_t)(8 * kLoadWaves) * ldw * 2;
    const auto load_tile = [&](int stage_off) {
      if (k0 == d0) {
        rows_of(d1);
        xb = uniform_ptr(reinterpret_cast<const char*>(x1));
      }
#pragma unroll
      for (int pc = 0; pc < kPieces; ++pc) {
        const lptr_t dst = lds3 + (stage_off + wave * 1024 + pc * kLoadWaves * 1024);     // x pieces fill the A tile, W pieces follow
        if (pc < kA) {
          asm("" : "+v"(offx[pc]));
          __builtin_amdgcn_global_load_lds(xb + offx[pc], dst, 16, 0, 0);
        } else {
          asm("" : "+v"(offW));
          __builtin_amdgcn_global_load_lds(wb + (pc - kA) * w_step + offW, dst, 16, 0, 0);
        }
      }
      k0 += BK;
      xb += kRowBytes;
      wb += kRowBytes;
    };
    // at most N newer k-tiles may still be on their way (loads complete in issue order)
    const auto wait_tiles = [&](int tiles) {
      if (tiles <= 0) wait_loads<0>();
      else if (tiles == 1) wait_loads<kPieces>();
      else if (kStages > 3 && tiles == 2) wait_loads<2 * kPieces % 64>();
      else if (kStages > 4 && tiles == 3) wait_loads<3 * kPieces % 64>();
      else if (kStages > 5 && tiles == 4) wait_loads<4 * kPieces % 64>();
      else if (kStages > 6 && tiles == 5) wait_loads<5 * kPieces % 64>();
      else wait_loads<(kStages - 1) * kPieces>();
    };
    // Where fragments are read a whole k-tile ahead, a stage is free one k-tile later: those reads may still be on their way when the
    // k-tile behind it is published.
    constexpr int kDepth = kStages - (S::kAhead > 1 ? 1 : 0);
    const int first = nk < kDepth ? nk : kDepth;
#pragma unroll
    for (int t = 0; t < kDepth; ++t)
      if (t < first) load_tile(t * S::kStage);
    wait_tiles(first - 1);
    meet();
    int to = kDepth == kStages ? 0 : kDepth * S::kStage, t = 0;
    for (; t + kDepth < nk; ++t) {                    // k-tile t + 1 has landed; every wave has read k-tile t + kDepth - kStages
      wait_loads<(kDepth - 2) * kPieces>();
      meet();
      load_tile(to);
      to = to + S::kStage == S::kLdsBytes ? 0 : to + S::kStage;
    }
    for (; t + 1 < nk; ++t) {
      wait_tiles(nk - 2 - t);
      meet();
    }
  }

  // A multiplying wave
  template <typename Start, typename Request>
  static __device__ __forceinline__ void multiply(const unsigned char* lds_base, int nk, int wave, int lane, f32x16 (&acc)[MI][NJ],
                                                  Start&& start, Request&& request) {
    constexpr int kAhead = S::kAhead, kBufs = kAhead + 1;
    const int wm = wave / S::WN, wn = wave % S::WN;
    struct Frag { bf16x8 x[MI], w[NJ]; };
    const int frow = lane & 31, fk = lane >> 5;
    // A fragment's place in a stage is kept in a register (opaque: the compiler would share parts of them and add twice for each
    // read); blocks of 32 rows have the same swizzle.
    int xo[4], wo[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      xo[ks] = lds_off(S::block_row(0, wm) + frow, ks * 2 + fk);
      wo[ks] = lds_off(S::block_col(0, wn) + frow, ks * 2 + fk) + S::kATile;
      asm("" : "+v"(xo[ks]), "+v"(wo[ks]));
    }
    const auto read = [&](int stage_off, int ks, Frag& f, int pc) {       // the W fragments first
      if (pc < NJ) f.w[pc] = *reinterpret_cast<const bf16x8*>(lds_base + stage_off + wo[ks] + pc * 32 * kRowBytes);
      else f.x[pc - NJ] = *reinterpret_cast<const bf16x8*>(lds_base + stage_off + xo[ks] + (pc - NJ) * S::WM * 32 * kRowBytes);
    };
    // the MFMAs of one step; extra(m) is issued right behind MFMA m (sched_barrier keeps the order)
    const auto mma = [&](const Frag& f, auto&& extra) {
#pragma unroll
      for (int m = 0; m < MI * NJ; ++m) {
        const int i = m / NJ, j = m % NJ;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.x[i], f.w[j], acc[i][j], 0, 0, 0);
        extra(m);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    const auto publish = [&] {
      if constexpr (kAhead == 1) __builtin_amdgcn_s_waitcnt(0xc07f);             // lgkmcnt(0): this wave's reads have returned
      meet();
    };
    start();
    meet();
    Frag f[kBufs];
#pragma unroll
    for (int s = 0; s < kAhead; ++s)
#pragma unroll
      for (int pc = 0; pc < MI + NJ; ++pc) read(0, s, f[s], pc);
    __builtin_amdgcn_sched_barrier(0);
    request();
    __builtin_amdgcn_sched_barrier(0);
    // k-tile t sits in the stage at `cur`, t + 1 in the one at `nxt`.  Before the step that first reads k-tile t + 1 it is
    // published; by then every wave's reads of tile t have returned.
    const auto tile = [&](int cur, int nxt, bool has_next) {
      // step s: its MFMAs, and between them the reads of the fragments kAhead steps on
      constexpr int kReads = MI + NJ, kPerMma = (kReads + MI * NJ - 1) / (MI * NJ);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        if (s == 4 - kAhead && has_next) publish();
        const bool ahead = s + kAhead >= 4;
        mma(f[s & (kBufs - 1)], [&](int m) {
          if (ahead && !has_next) return;
#pragma unroll
          for (int e = m * kPerMma; e < (m + 1) * kPerMma && e < kReads; ++e)
            read(ahead ? nxt : cur, (s + kAhead) & 3, f[(s + kAhead) & (kBufs - 1)], e);
        });
      }
    };
    int cur = 0, nxt = S::kStage;
    for (int t = 0; t + 1 < nk; ++t) {
      tile(cur, nxt, true);
      cur = nxt;
      nxt = nxt + S::kStage == S::kLdsBytes ? 0 : nxt + S::kStage;
    }
    tile(cur, nxt, false);
    settle_accumulators(acc);
  }

  template <typename Start, typename Request>
  static __device__ __forceinline__ void run(unsigned char* lds_base, const bf16_t* __restrict__ x0, int d0,
                                             const bf16_t* __restrict__ x1, int d1, const bf16_t* __restrict__ W, int ldw,
                                             int last, f32x16 (&acc)[MI][NJ], Start&& start, Request&& request) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nk = (d0 + d1) / BK;
    if (wave < kMulWaves) {
      multiply(lds_base, nk, wave, lane, acc, start, request);
    } else if (wave < kMulWaves + kLoadWaves) {
      load(lds_base, x0, d0, x1, d1, W, ldw, last, wave - kMulWaves, lane);
      request();
    } else {
      meet();
      request();
      for (int t = 0; t + 1 < nk; ++t) meet();
    }
  }
};

}  // namespace aquakv

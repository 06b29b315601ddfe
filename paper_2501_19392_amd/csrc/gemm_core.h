// What the bf16 main loops of the linear predictors (Sect. 3.2 of the AQUA-KV paper) share: operand types, the swizzled LDS layout of a
// k-tile, the order of tiles over the XCDs and the end of a loop.  (Loops: gemm_tile.h, gemm_two_heads.h, gemm_token_slab.h, gemm_team.h.)
//
// v_mfma_f32_32x32x16_bf16, fp32 accumulate.  Both operands are K-contiguous (x is [T, K],
// W is [D, K]), so A and B fragments are 128-bit LDS reads.  Every output accumulates K in
// ascending order in one accumulator, whatever the tile and the number of rows in the call: a row's
// prediction does not depend on its neighbours, which is what lets decode reproduce encode.
//
// Inside a 32 x 32 block of accumulators the lane holds column lane % 32 and rows 8 b + 4 (lane / 32) + r in register 4 b + r.
//
// Operands go from global memory straight into LDS (global_load_lds_dwordx4): no staging
// registers, no ds_write instructions.  One such instruction of a wave fills 1 KiB of LDS,
// lane l at byte 16 l, i.e. 8 consecutive tile rows with lane l -> row l/8, slot l%8.  The LDS
// layout is swizzled (lds_off), so the lane fetches from global memory the chunk that belongs
// in its slot.  The compiler does not track these writes to LDS: completion is awaited with an
// explicit vmcnt before the barrier that publishes a k-tile (loads complete in issue order, so
// waiting until at most n tiles' worth are outstanding means every older tile has landed).
#pragma once
#include "device_utils.h"

namespace aquakv {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8;

constexpr int BM = 256, BN = 128, BK = 64;       // block tile
constexpr int kRowBytes = BK * 2;                // 128 B of bf16 per LDS row
constexpr int kATileBytes = BM * kRowBytes;      // 32 KiB
constexpr int kBTileBytes = BN * kRowBytes;      // 16 KiB
constexpr int kStageBytes = kATileBytes + kBTileBytes;   // 48 KiB
constexpr int kStages = 3;                       // LDS ring of k-tiles
constexpr int kMainLoopLdsBytes = kStages * kStageBytes;
// After the last MFMA of a main loop: its results reach the accumulators 8 passes (32 cycles) later, and vector instructions
// that read them sooner see old values.  The compiler keeps 12 wait states there, but not on every path: where a branch and its
// other side meet again before the first read, it counts them on one of the two sides only.  Seen with ROCm 7.2 in the scoring
// kernels of the round-to-nearest backbone on tiles of 32 rows without a bias (fused_tile_kernel<2 or 4, kTileScores, 1, ..>):
// s_cmp, v_and, s_cbranch, v_mov, s_nop 0 between the last MFMA and the first v_accvgpr_read, 5 states, the longer side being
// the one that loads the bias.  So every main loop ends with the states spelled out.  An empty asm statement per block takes one
// of its values first: nothing else keeps the MFMAs, which touch no memory, from sinking past the wait into a later block.
__device__ __forceinline__ void tie_accumulators(const f32x16& acc) { asm volatile("" ::"v"(acc[0])); }
template <typename T, int N> __device__ __forceinline__ void tie_accumulators(const T (&acc)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) tie_accumulators(acc[i]);
}
template <typename T> __device__ __forceinline__ void settle_accumulators(const T& acc) {
  __builtin_amdgcn_sched_barrier(0);
  tie_accumulators(acc);
  asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// 16-byte chunk `ch` (0..7) of LDS row `row`.  A row is 128 B = half of the 64 banks, so even
// and odd rows already sit in different bank halves; the chunk is XOR-swizzled with row/2 so
// that the 16 lanes served together by a 128-bit fragment read (16 consecutive rows, same
// chunk) touch all 64 banks exactly once.
__device__ __forceinline__ int lds_off(int row, int ch) { return row * kRowBytes + ((ch ^ ((row >> 1) & 7)) << 4); }

// XCD-aware tile order: consecutive workgroup ids land on different XCDs, so
// give each XCD a contiguous range of tiles (n fastest): the column tiles of
// a row tile then share that XCD's L2 copy of the x rows.
__device__ __forceinline__ int remap_block(int bid, int nblocks) {
  constexpr int kXcd = 8;
  if (nblocks % kXcd != 0) return bid;
  return (bid % kXcd) * (nblocks / kXcd) + bid / kXcd;
}

}  // namespace aquakv

// bf16 MFMA main loop of the linear predictors (Sect. 3.2 of the AQUA-KV paper) on a tile of 64 token rows x ALL 1024
// outputs (8 kv heads x 128), for eight wavefronts: wave h owns head h.  This is the shape the encoder needs when the
// rotation group is the whole token (Sect. 4.1: groups of 1024): scale and the butterfly stages across the heads want
// all 8 heads of a token in one workgroup.
//
// Same instruction (v_mfma_f32_32x32x16_bf16), operand orientation and K order per output as gemm_core.h, hence the
// same bits.  Every workgroup streams the whole of W from L2, and each row of W is multiplied by one wave only, so W does not
// go through LDS: a wave loads its fragments straight into registers, three steps of 16 k ahead, from a re-tiled copy
// (retile_w_kernel in fused_wide_encode.hip writes it into the call's workspace; a few microseconds for 2 - 4 MiB) that
// holds them in the order of use, 1 KiB of consecutive bytes per fragment.  Only the 64 token rows (8 KiB per k-tile of 64)
// are shared by the waves and staged in LDS.  Bound by what a CU takes from L2: 32 KiB of W per step of 16 k at some 57
// bytes per cycle are 575 cycles, against 512 cycles of matrix work for the two waves of a SIMD.  (With W staged in LDS the
// loop took 2560 cycles per 32 k.)
#pragma once
#include "gemm_core.h"

namespace aquakv {

constexpr int kSlabRows = 64;                          // token rows of a tile
constexpr int kSlabCols = 1024;                        // outputs of a tile = 8 heads x 128
constexpr int kSlabWaves = 8;
constexpr int kSlabStageBytes = kSlabRows * kRowBytes; // 8 KiB: a k-tile of 64 of the token rows
constexpr int kSlabStages = 4;
constexpr int kSlabLdsBytes = kSlabStages * kSlabStageBytes;
constexpr int kSlabStepBytes = kSlabCols * 16 * 2;     // W of one step of 16 k in the re-tiled copy
// Byte of the 16-byte chunk of W row `row` (0..1023), inputs 8 chunk ... + 7, in the re-tiled copy: fragment
// (step = chunk / 2, head, block of 32 rows), lane = row % 32 + 32 (chunk % 2).
__host__ __device__ constexpr int64_t slab_w_off(int row, int chunk) {
  return (int64_t)(chunk >> 1) * kSlabStepBytes + (row >> 5) * 1024 + ((row & 31) + 32 * (chunk & 1)) * 16;
}

// acc[i][j]: the 32 x 32 block at token rows 32 i, outputs 128 wave + 32 j of the tile; inside it the lane holds output
// column lane % 32 and rows 8 blk + 4 (lane / 32) + r in register 4 blk + r (as gemm_core.h).
// `lds_base` points at kSlabLdsBytes bytes of LDS.  The caller puts a barrier before it reuses the LDS.  Requires
// K = d0 + d1 a multiple of 128, d0 of 64.  `Wt`: the re-tiled copy of the 1024 x K weights.
//
// Schedule.  k-tile t of the token rows lives in stage t % 4; wave w loads its rows 8 w ... (one instruction per k-tile), two
// k-tiles ahead.  A k-tile is four steps; in step s:
//   MFMAs (t, s)   + reads of the row fragments of the next step   + loads of the W fragments three steps ahead
// and before step 3 the barrier that publishes k-tile t + 1.
__device__ __forceinline__ void gemm_mainloop_token_slab(unsigned char* lds_base, const bf16_t* __restrict__ x0, int d0,
                                                         const bf16_t* __restrict__ x1, int d1,
                                                         const bf16_t* __restrict__ Wt, int64_t T, int64_t m0,
                                                         f32x16 (&acc)[2][4]) {
  typedef __attribute__((address_space(3))) unsigned char* lptr_t;
  typedef const __attribute__((address_space(1))) char* gptr_t;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int K = d0 + d1, nk = K / BK, nsteps = K / 16;

  // one load instruction of a wave fills 1 KiB of LDS = 8 token rows of 128 B, swizzled as in gemm_core.h
  const int last = (int)((T - 1 - m0) < (kSlabRows - 1) ? (T - 1 - m0) : (kSlabRows - 1));
  const int row = tid >> 3, rowc = row < last ? row : last;
  const int ch16 = ((tid & 7) ^ ((tid >> 4) & 7)) * 16;
  const auto uniform_ptr = [](const char* p) {
    const uint64_t u = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
    return (gptr_t)(((uint64_t)hi << 32) | lo);
  };
  const lptr_t lds3 = (lptr_t)lds_base;
  auto load_rows = [&](int kt) {
    const int k0 = kt * BK;
    const bool second = k0 >= d0;
    const int ld2 = __builtin_amdgcn_readfirstlane((second ? d1 : d0) * 2);
    const gptr_t base = uniform_ptr(reinterpret_cast<const char*>(second ? x1 : x0) +
                                    (m0 * ld2 + (int64_t)(second ? k0 - d0 : k0) * 2));
    __builtin_amdgcn_global_load_lds(base + ((uint32_t)__umul24(rowc, ld2) + ch16),
                                     lds3 + ((kt & (kSlabStages - 1)) * kSlabStageBytes + wave * 1024), 16, 0, 0);
  };
  const uint32_t offW = (uint32_t)(wave * 4096 + lane * 16);
  struct WFrag { bf16x8 v[4]; };
  auto load_w = [&](int step, WFrag& f) {
    const gptr_t base = uniform_ptr(reinterpret_cast<const char*>(Wt) + (int64_t)step * kSlabStepBytes);
#pragma unroll
    for (int j = 0; j < 4; ++j) f.v[j] = *reinterpret_cast<const __attribute__((address_space(1))) bf16x8*>(base + offW + j * 1024);
  };
  const int frow = lane & 31, fk = lane >> 5;
  struct XFrag { bf16x8 v[2]; };
  auto read_x = [&](int kt, int ks, XFrag& f) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
      f.v[i] = *reinterpret_cast<const bf16x8*>(lds_base + (kt & (kSlabStages - 1)) * kSlabStageBytes + lds_off(i * 32 + frow, ks * 2 + fk));
  };
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  auto meet = [&] {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };

  load_rows(0);
  load_rows(1);                                        // nk >= 2
  __builtin_amdgcn_sched_barrier(0);                   // (the count below wants them older than the fragment loads)
  WFrag w[4];
  load_w(0, w[0]);
  load_w(1, w[1]);
  load_w(2, w[2]);
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0x0f70 | 12);             // vmcnt(12): both k-tiles of this wave's rows have landed
  meet();
  XFrag x[2];
  read_x(0, 0, x[0]);
  __builtin_amdgcn_sched_barrier(0);

  for (int t = 0; t < nk; ++t) {
    if (t + 2 < nk) load_rows(t + 2);                  // its stage held k-tile t - 2, read by all before the last barrier
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if (s == 3 && t + 1 < nk) {
        // Publish k-tile t + 1.  This wave's rows of it were requested a k-tile ago, before 16 of the fragment loads issued
        // since; at most 12 of those (three steps) and the rows of t + 2 may still be out.
        __builtin_amdgcn_s_waitcnt(0x0070 | 13);       // vmcnt(13) lgkmcnt(0)
        meet();
      }
      const int step = 4 * t + s;
      const WFrag& wf = w[s];
      const XFrag& xf = x[s & 1];
      if (s < 3) read_x(t, s + 1, x[(s + 1) & 1]);
      else if (t + 1 < nk) read_x(t + 1, 0, x[0]);
      // (behind the last step the loads repeat it: the count of loads in flight stays the same)
      load_w(step + 3 < nsteps ? step + 3 : nsteps - 1, w[(s + 3) & 3]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf.v[i], wf.v[j], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  settle_accumulators();
}

}  // namespace aquakv

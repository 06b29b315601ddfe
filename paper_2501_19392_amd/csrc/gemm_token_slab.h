// bf16 MFMA main loop of the linear predictors (Sect. 3.2 of the AQUA-KV paper) on a tile of 64 token rows x ALL 1024
// outputs (8 kv heads x 128), for eight wavefronts: wave h owns head h.  This is the shape the encoder needs when the
// rotation group is the whole token (Sect. 4.1: groups of 1024): scale and the butterfly stages across the heads want
// all 8 heads of a token in one workgroup.
//
// Same instruction (v_mfma_f32_32x32x16_bf16), operand orientation and K order per output as gemm_core.h, hence the
// same bits.  Every workgroup streams the whole of W, and each row of W is multiplied by one wave only: a wave loads its own
// fragments, kSlabAhead steps of 16 k ahead, from a re-tiled copy (retile_w_kernel in fused_wide_encode.hip writes it into the
// call's workspace; a few microseconds for 2 - 4 MiB) that holds them in the order of use, 1 KiB of consecutive bytes per
// fragment.  Half of them go straight to registers, the other half to a ring of its own in LDS, because neither has room for
// what must be in flight: the workgroups of an XCD walk W in step, so every step waits for L2 to fetch it once (some 2700
// cycles), and 57 bytes per cycle into a CU over that time are 150 KiB.  Only the 64 token rows (8 KiB per k-tile of 64) are
// shared by the waves.  Three steps ahead in registers alone: 1000 cycles per step; two k-tiles of 32 through LDS: 1280.
// The matrix work of the two waves of a SIMD is 512 cycles per step, 32 KiB at 57 bytes per cycle 575.
#pragma once
#include "gemm_core.h"

namespace aquakv {

constexpr int kSlabRows = 64;                          // token rows of a tile
constexpr int kSlabCols = 1024;                        // outputs of a tile = 8 heads x 128
constexpr int kSlabWaves = 8;
constexpr int kSlabStageBytes = kSlabRows * kRowBytes; // 8 KiB: a k-tile of 64 of the token rows
constexpr int kSlabStages = 3;
constexpr int kSlabAhead = 6;                          // steps of 16 k between the request of a W fragment and its use
constexpr int kSlabSlots = kSlabAhead + 1;             // ring of W fragments in LDS, per wave: 2 KiB a step
constexpr int kSlabRingBytes = kSlabSlots * 2048;
constexpr int kSlabLdsBytes = kSlabStages * kSlabStageBytes + kSlabWaves * kSlabRingBytes;      // 136 KiB
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
// Schedule.  k-tile t of the token rows lives in stage t % 3; wave w loads its rows 8 w ... (one instruction per k-tile), two
// k-tiles ahead.  A k-tile is four steps; in step s:
//   MFMAs (t, s)   + LDS reads of the next step's fragments   + requests of the W fragments kSlabAhead steps ahead
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
  auto load_rows = [&](int kt, int stage_off) {
    const int k0 = kt * BK;
    const bool second = k0 >= d0;
    const int ld2 = __builtin_amdgcn_readfirstlane((second ? d1 : d0) * 2);
    const gptr_t base = uniform_ptr(reinterpret_cast<const char*>(second ? x1 : x0) +
                                    (m0 * ld2 + (int64_t)(second ? k0 - d0 : k0) * 2));
    __builtin_amdgcn_global_load_lds(base + ((uint32_t)__umul24(rowc, ld2) + ch16), lds3 + (stage_off + wave * 1024), 16, 0, 0);
  };
  // W of a step: blocks 0, 1 of this wave's head to LDS (the wave's ring), blocks 2, 3 to registers, in this order: when the
  // registers have arrived, so have the LDS ones (loads complete in issue order)
  const uint32_t offW = (uint32_t)(wave * 4096 + lane * 16);
  const int ring0 = kSlabStages * kSlabStageBytes + wave * kSlabRingBytes;
  struct WRegs { bf16x8 v[2]; };
  auto load_w = [&](int step, int slot_off, WRegs& f) {
    const gptr_t base = uniform_ptr(reinterpret_cast<const char*>(Wt) + (int64_t)step * kSlabStepBytes);
#pragma unroll
    for (int j = 0; j < 2; ++j)
      __builtin_amdgcn_global_load_lds(base + (offW + (uint32_t)(j * 1024)), lds3 + (ring0 + slot_off + j * 1024), 16, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 2; ++j)
      f.v[j] = *reinterpret_cast<const __attribute__((address_space(1))) bf16x8*>(base + offW + (2 + j) * 1024);
    __builtin_amdgcn_sched_barrier(0);
  };
  const int frow = lane & 31, fk = lane >> 5;
  struct XFrag { bf16x8 v[2]; };
  auto read_x = [&](int stage_off, int ks, XFrag& f) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
      f.v[i] = *reinterpret_cast<const bf16x8*>(lds_base + stage_off + lds_off(i * 32 + frow, ks * 2 + fk));
  };
  auto read_w = [&](int slot_off, WRegs& f) {
#pragma unroll
    for (int j = 0; j < 2; ++j) f.v[j] = *reinterpret_cast<const bf16x8*>(lds_base + ring0 + slot_off + j * 1024 + lane * 16);
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
  const auto next_slot = [](int s) { return s + 2048 == kSlabRingBytes ? 0 : s + 2048; };

  load_rows(0, 0);
  load_rows(1, kSlabStageBytes);                       // nk >= 2
  __builtin_amdgcn_sched_barrier(0);                   // (the counts below want them older than the fragment loads)
  WRegs w[8];                                          // registers of step n: w[n % 8]
#pragma unroll
  for (int n = 0; n < kSlabAhead; ++n) load_w(n < nsteps ? n : nsteps - 1, n * 2048, w[n]);      // nsteps >= 8
  __builtin_amdgcn_s_waitcnt(0x0f70 | ((4 * (kSlabAhead - 1)) & 15) | (((4 * (kSlabAhead - 1)) >> 4) << 14));   // rows and step 0 have landed
  meet();
  XFrag x[2];
  WRegs wl[2];
  int cur = 0, nxt = kSlabStageBytes, far = 2 * kSlabStageBytes;      // stages of k-tiles t, t + 1, t + 2
  int read_slot = 0, load_slot = kSlabAhead * 2048;
  read_x(cur, 0, x[0]);
  read_w(read_slot, wl[0]);
  __builtin_amdgcn_sched_barrier(0);

  for (int t2 = 0; t2 < nk; t2 += 2) {                 // two k-tiles = eight steps at a time (nk is even)
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int t = t2 + (u >> 2), s = u & 3, step = 4 * t2 + u;
      const auto mma = [&](int m) {
        const int i = m & 1, j = m >> 1;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[u & 1].v[i], j < 2 ? wl[u & 1].v[j] : w[u].v[j - 2], acc[i][j], 0, 0, 0);
      };
      // The memory work of a step goes behind its first two MFMAs: the compiler waits for every outstanding LDS read before
      // the first of them (it cannot count reads beside direct-to-LDS loads), so none for the next step may be out by then.
      mma(0);
      mma(1);
      __builtin_amdgcn_sched_barrier(0);
      // (the stage of k-tile t + 2 held k-tile t - 1: every wave had its last reads back before k-tile t was published)
      if (s == 0 && t + 2 < nk) load_rows(t + 2, far);
      // (behind the last step the loads repeat it: the count of loads in flight stays the same)
      load_w(step + kSlabAhead < nsteps ? step + kSlabAhead : nsteps - 1, load_slot, w[(u + kSlabAhead) & 7]);
      load_slot = next_slot(load_slot);
      // The next step's fragments have landed when at most the loads of the kSlabAhead - 1 steps behind it are out (4 each).
      // In step 3 that covers this wave's rows of k-tile t + 1 as well: requested seven steps ago, they are older.
      __builtin_amdgcn_s_waitcnt(0x0f70 | ((4 * (kSlabAhead - 1)) & 15) | (((4 * (kSlabAhead - 1)) >> 4) << 14));
      asm volatile("" ::: "memory");
      read_slot = next_slot(read_slot);
      if (s == 3 && t + 1 < nk) {
        meet();                                        // (its reads of k-tile t returned before the MFMAs above)
        read_x(nxt, 0, x[(u + 1) & 1]);
        const int old = cur;
        cur = nxt; nxt = far; far = old;
      } else if (s < 3) {
        read_x(cur, s + 1, x[(u + 1) & 1]);
      }
      read_w(read_slot, wl[(u + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int m = 2; m < 8; ++m) mma(m);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // the repeated loads of the last steps may still be on their way into the rings, which the caller is about to reuse
  __builtin_amdgcn_s_waitcnt(0x0f70);
  settle_accumulators(acc);
}

}  // namespace aquakv

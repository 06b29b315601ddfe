// Fused predictor kernels (Alg. "encode" / "decode" of the AQUA-KV paper: predictor of Sect. 3.2, backbone of Sect. 2) on
// tiles of 32, 64, 96, 128, 192 or 320 token rows x one kv head (which one: tile_rows in fused_kernels.hip).
//
// Same main-loop bits (gemm_tile.h), same group bodies, hence the same results.  Only the four multiplying waves hold accumulators; the
// epilogue parks them in LDS, all rows where they fit (else 256), and all waves work on them, 16 groups per wave and pass, one
// group per quad of lanes; on tiles of 32 and 64 rows, which would
// leave half of the waves (32 rows) or one of two per SIMD (64) idle, 8 groups per wave, one group per eight lanes.  A wave alone
// on its SIMD is bound by latency, so the work per lane is what counts: keys and values of 128 tokens, 16-point grid, 22.9 -> 20.8 us
// (256 points: 29.8 -> 25.1), decode of 1100 tokens with groups across the heads 27.7 -> 24.4 (those with the main loops before: now 17.1 and
// 21.3).  The encoder's epilogue is bound by vector issue, 41 to 44 instructions a value.  Codes turned back by further waves
// during the main loop gained nothing: their LDS reads hold up the operands' (4000 tokens across the heads 34.5 -> 48 us).
// On 96 and 192 rows three waves share a SIMD, 168 registers each: with 16 values per lane and four sub-vectors searched at a time the quantizer takes
// 105; with eight at a time it spilled (3072 tokens 35.4 us against 39.6; 64 points 38.2 against 45.6).
#pragma once
#include "attend_piece.h"
#include "fused_epilogue.h"
#include "gemm_tile.h"
#include "kernels.h"

namespace aquakv {

enum TileMode : int { kTileEncode = 0, kTileDecode = 1, kTileScores = 2, kTilePredict = 3 };

struct XcdSplit { int log2_n, even; uint32_t per_heads, per_all; };   // xcd_split

struct TileArgs {
  const bf16_t* x0;
  const bf16_t* x1;
  const bf16_t* W;
  const float* bias;
  const int8_t* signs;
  const float* codebook;
  const uint32_t* table;
  const bf16_t* X;
  uint8_t* codes;
  uint16_t* scales;
  bf16_t* Xhat;
  Prediction P;                   // kTilePredict
  const bf16_t* q;
  const float* rope_cos;
  const float* rope_sin;
  float* scores;
  float score_scale;
  int d0, d1, D, q_heads;
  int seq_len;                    // rows per sequence (one sequence: all rows)
  int tiles_per_seq;              // tiles never straddle sequences
  int ldw;                        // row stride of W
  // sums of a product over the first part of its inputs, in two halves of 16 bits, [T, D] each
  uint16_t* sums_hi;
  uint16_t* sums_lo;
  XcdSplit xcd;                   // tile_of
};
// Two products in one launch: the first `blocks` workgroups work on job[0], the others on job[1], or (tiles of 32 rows) store the
// sums of job[1] and nothing else if it has a place for them.
struct TilePair {
  TileArgs job[2];
  int blocks;
};
// Job 0 on tiles of MB0 row blocks, job 1 on tiles of MB1
template <int MB0, int MB1> struct TwoTiles {
  static constexpr int kWaves = Tile<MB0>::kWaves > Tile<MB1>::kWaves ? Tile<MB0>::kWaves : Tile<MB1>::kWaves;
};
// What is done about sums: nothing, the product goes on from those that are there, or `keep` says whether they alone are wanted.
enum TileSums : int { kNoSums = 0, kUseSums = 1, kKeepSums = 2 };
// Decode of one or two tensors (job[1] has `tiles` - pair.blocks workgroups) and, on the workgroups behind them, pieces of the attention of
// a layer recovered before.
struct TileAttend {
  TilePair pair;
  int tiles;
  AttendCacheArgs attend;
};
// Which tile a workgroup works on.  Consecutive workgroups go to consecutive XCDs, each with an L2 of its own that fetches the x rows and
// the rows of W of its tiles once.  The row blocks are split into 8 / n groups and the heads into n, one of each to an XCD: the n that
// fetches least.  Row blocks that do not come out even follow in the plain order.  1024
// tokens on 32 rows: n = 2, 768 rows of 128 bytes per k-tile and XCD where heads in the plain order fetch 1152.  (Row blocks that come out
// even only with n = 8 must not be split so: 9000 tokens on 320 rows 68 -> 80 us.)
// n = 1 << log2_n; even: row blocks in the split; per_x: ceil(2^32 / x), 0 for one: a division is some 20 instructions ahead of
// everything else (flush of 128 tokens 17.5 -> 17.1 us without the seven that were here).
inline XcdSplit xcd_split(int64_t row_blocks, int H, int rows) {
  XcdSplit best = {0, 0, 0, 0};
  int64_t least = 0;
  for (int l = 0; l < 4; ++l) {
    const int n = 1 << l;
    const int64_t even = row_blocks / (8 / n) * (8 / n), rest = row_blocks - even;
    const int64_t fetched = (even * n / 8 + rest) * rows + (H / n + (rest != 0)) * kGroup;
    if (H % n == 0 && even != 0 && (best.even == 0 || fetched < least)) { best = {l, (int)even, 0, 0}; least = fetched; }
  }
  const auto per = [](uint32_t d) { return d == 1 ? 0u : (uint32_t)(((1ull << 32) + d - 1) / d); };
  best.per_heads = per(H >> best.log2_n);
  best.per_all = per(H);
  return best;
}
__device__ __forceinline__ void tile_of(int block, int H, const XcdSplit& s, int& tile_m, int& head) {
  const bool plain = block >= s.even * H;
  const int i = plain ? block : block >> 3, heads = plain ? H : H >> s.log2_n, xcd = plain ? 0 : block & 7;
  const uint32_t per = plain ? s.per_all : s.per_heads;
  const int slot = per == 0 ? i : (int)__umulhi((uint32_t)i, per);          // i / heads, exact while i * heads < 2^32
  const int n_rows = plain ? 1 : 8 >> s.log2_n, group = xcd & ((1 << s.log2_n) - 1);
  head = group * heads + (i - slot * heads);
  tile_m = slot * n_rows + (xcd >> s.log2_n);
}
// How an epilogue splits a tile, and the LDS it takes
template <int MODE, int MB> struct TileEpilogue {
  using S = Tile<MB>;
  static constexpr int kVals = MB <= 3 || MB == 6 ? 16 : kValsPerLane;            // values of a group per lane
  static constexpr int kWaveRows = kVals / 2;                          // groups per wave and pass
  static constexpr int kPassRows = S::kRows < kWaveRows * S::kWaves ? S::kRows : kWaveRows * S::kWaves;
  static constexpr int kPasses = (S::kRows + kPassRows - 1) / kPassRows;
  // Rows parked at a time: all of them where the LDS has room.  (What is not parked stays in the multiplying waves' registers.)
  static constexpr int kParkPasses = kPasses < 3 ? kPasses : 2, kParkRows = kParkPasses * kPassRows;
  static constexpr int kParkBlocks = MB < 9 ? MB : 8;              // predictions: row blocks parked at a time
  static constexpr int kBytes = MODE != kTilePredict ? (int)sizeof(Lds) + kParkRows * kLdP * 4 : kParkBlocks * 32 * kLdP * 4;
  static_assert(kBytes <= 160 * 1024, "LDS of one CU");
  static constexpr int kLdsBytes = kBytes > S::kLdsBytes ? kBytes : S::kLdsBytes;
};
// workgroup `block` of those that work on `a`, of WAVES waves; smem: TileEpilogue<MODE, MB>::kLdsBytes of LDS
template <int NCW, int MODE, int MB, bool WIDE, int SUMS, int WAVES = Tile<MB>::kWaves>
__device__ __forceinline__ void fused_tile(const TileArgs& a, int block, bool keep, unsigned char* smem) {
  using S = Tile<MB>;
  static_assert(WAVES == S::kWaves || (MODE == kTilePredict && WAVES > S::kWaves), "an epilogue is split over the tile's own number of waves");
  static_assert(!WIDE || MODE != kTileEncode, "the quantizer needs the whole group: groups across the heads are not fused");
  using E = TileEpilogue<MODE, MB>;
  constexpr int kVals = E::kVals, kWaveRows = E::kWaveRows, kPassRows = E::kPassRows, kPasses = E::kPasses;
  constexpr bool kEpilogue = MODE != kTilePredict;
  Lds& cl = *reinterpret_cast<Lds*>(smem);                      // grid and table at the start of the LDS (codec_core.h)
  float* const park = reinterpret_cast<float*>(smem + sizeof(Lds));

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int H = a.D / kGroup;
  int tile_m, head;
  tile_of(block, H, a.xcd, tile_m, head);
  const int b = tile_m < a.tiles_per_seq ? 0 : tile_m / a.tiles_per_seq, t0 = (tile_m - b * a.tiles_per_seq) * S::kRows;
  const int left = a.seq_len - t0;
  const int n_rows = left < S::kRows ? left : S::kRows;         // valid rows of this tile
  const int64_t m0 = (int64_t)b * a.seq_len + t0;               // its first row
  const int n0 = head * kGroup;
  const int q = group_pos<kVals>(lane), wrow = lane / (kGroup / kVals);      // position in the group, group of the wave

  // What the epilogue reads from memory is requested from inside the main loop (by multiplying waves behind their first fragments, by loading
  // waves behind their last loads) and waits in registers.
  constexpr bool kEnc = MODE == kTileEncode;
  constexpr bool kWideGrid = WIDE && !is_rtn(NCW) && kEpilogue;
  // Codes of 8 heads x 16 bytes beside a wave's 160 accumulators and 56 registers of fragments spilled: requested behind the main loop (10000
  // tokens, 256 points 92.5 -> 91.6 us).
  constexpr bool kLate = kWideGrid && NCW == 256 && MB == 10;
  struct In { u32x4 x[kEnc ? kVals / 8 : 1]; CodeWords w; };
  // several passes: the inputs of the first are requested from inside the main loop, those of each next one during the one before
  In in[2];
  WideCodes<NCW> wide[kWideGrid ? 2 : 1];
  float cb_a = 0.f, cb_b = 0.f;
  TableRegs<S::kThreads> table_regs;
  const bool use_table = kEnc && !is_rtn(NCW) && a.table != nullptr;
  constexpr int kGridPoints = is_rtn(NCW) || !kEpilogue ? 0 : NCW;
  static_assert(kGridPoints <= S::kThreads, "one grid point per thread");
  u32x2 qreg = {0, 0};
  const int rep = MODE == kTileScores ? a.q_heads / H : 0;
  const auto fetch = [&](int h) {
    const int lrow = h * kPassRows + wave * kWaveRows + wrow;
    const int64_t row = m0 + (lrow < n_rows ? lrow : n_rows - 1);
    if constexpr (kEnc) {
      const u32x4* src = reinterpret_cast<const u32x4*>(a.X + row * a.D + n0 + q * kVals);
#pragma unroll
      for (int k = 0; k < kVals / 8; ++k) in[h & 1].x[k] = src[k];
    } else {
      in[h & 1].w = request_words<NCW, WIDE, kVals>(a.codes, a.scales, row * H + head, q);
      if constexpr (kWideGrid) request_wide_codes<NCW, kVals>(a.codes, row, q, wide[h & 1]);
    }
  };
  const int wm = wave / S::WN, wn = wave % S::WN;                // (of the multiplying waves)
  f32x16 acc[S::MI][S::NJ];
  const int frow = lane & 31, fk = lane >> 5;
  // element of [T, D] in register r of block (i, j)
  const auto sum_at = [&](int i, int j, int r) {
    const int lrow = S::block_row(i, wm) + (r >> 2) * 8 + fk * 4 + (r & 3);
    return (m0 + (lrow < n_rows ? lrow : n_rows - 1)) * a.D + n0 + S::block_col(j, wn) + frow;
  };
  uint16_t hi[S::MI][S::NJ][16], lo[S::MI][S::NJ][16];
  if constexpr (SUMS == kUseSums) {
    if (wave < kMulWaves) {
#pragma unroll
      for (int i = 0; i < S::MI; ++i)
#pragma unroll
        for (int j = 0; j < S::NJ; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) { hi[i][j][r] = a.sums_hi[sum_at(i, j, r)]; lo[i][j][r] = a.sums_lo[sum_at(i, j, r)]; }
    }
  }

  const int ldw = SUMS == kNoSums ? a.d0 + a.d1 : a.ldw;
  TileLoop<MB>::run(smem, a.x0 + m0 * a.d0, a.d0, a.d1 ? a.x1 + m0 * a.d1 : a.x1, a.d1, a.W + (int64_t)n0 * ldw, ldw, n_rows - 1, acc, [&] {
#pragma unroll
    for (int i = 0; i < S::MI; ++i)
#pragma unroll
      for (int j = 0; j < S::NJ; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          acc[i][j][r] = SUMS == kUseSums ? __uint_as_float(((uint32_t)hi[i][j][r] << 16) | lo[i][j][r]) : 0.f;
  }, [&] {
    if (kEpilogue && !(SUMS == kKeepSums && keep)) {
      if ((int)threadIdx.x < kGridPoints) { cb_a = a.codebook[2 * threadIdx.x]; cb_b = a.codebook[2 * threadIdx.x + 1]; }
      if (use_table) table_regs.request(a.table);
      if constexpr (MODE == kTileScores) {
        // the queries of this head (at most 8 x 128, adjacent in memory), 4 values per thread
        if ((int)threadIdx.x * 4 < rep * kGroup)
          qreg = *reinterpret_cast<const u32x2*>(a.q + ((int64_t)b * a.q_heads + head * rep) * kGroup + threadIdx.x * 4);
      }
      if (!kLate && wave * kWaveRows < kPassRows) fetch(0);
    }
  });
  if constexpr (kLate) fetch(0);
  if (SUMS == kKeepSums && keep) {
    if (wave < kMulWaves) {
#pragma unroll
      for (int i = 0; i < S::MI; ++i)
#pragma unroll
        for (int j = 0; j < S::NJ; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const uint32_t u = __float_as_uint(acc[i][j][r]);
            if (S::block_row(i, wm) + (r >> 2) * 8 + fk * 4 + (r & 3) < n_rows) {
              a.sums_hi[sum_at(i, j, r)] = (uint16_t)(u >> 16);
              a.sums_lo[sum_at(i, j, r)] = (uint16_t)u;
            }
          }
    }
    return;
  }

  float bv[S::NJ];
#pragma unroll
  for (int j = 0; j < S::NJ; ++j) bv[j] = a.bias != nullptr && wave < kMulWaves ? a.bias[n0 + S::block_col(j, wn) + frow] : 0.f;

  if constexpr (!kEpilogue) {
    // Parked and stored by all waves, 512 bytes of a row per half wave: the multiplying waves alone store 4 bytes a lane.
    float* const rows = reinterpret_cast<float*>(smem);
    float* const out = (n0 < a.P.split ? a.P.first + n0 : a.P.second + (n0 - a.P.split)) + frow * 4;
#pragma unroll
    for (int first = 0; first < MB; first += E::kParkBlocks) {
      __syncthreads();                                          // the ring, or the rows before, have been read
      if (wave < kMulWaves) {
#pragma unroll
        for (int i = first / S::WM; i < S::MI && i * S::WM < first + E::kParkBlocks; ++i)
#pragma unroll
          for (int j = 0; j < S::NJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
              rows[(S::block_row(i, wm) - first * 32 + (r >> 2) * 8 + fk * 4 + (r & 3)) * kLdP + S::block_col(j, wn) + frow] = acc[i][j][r] + bv[j];
      }
      __syncthreads();
      const int here = (MB - first < E::kParkBlocks ? MB - first : E::kParkBlocks) * 32;
      for (int row = wave * 2 + fk; row < here && first * 32 + row < n_rows; row += 2 * WAVES)
        *reinterpret_cast<f32x4*>(out + (m0 + first * 32 + row) * a.P.stride) = *reinterpret_cast<const f32x4*>(rows + row * kLdP + frow * 4);
    }
    return;
  } else {
    float sf[kVals] = {};
    if constexpr (!is_rtn(NCW)) load_signs(a.signs, head, q, sf);
    float* const q_lds = reinterpret_cast<float*>(cl.table);    // (no cell table in scores mode)
    __syncthreads();                                            // every wave is done reading the ring
    if ((int)threadIdx.x < kGridPoints)
      cl.cb[threadIdx.x] = make_float4(cb_a, cb_b, -0.5f * (cb_a * cb_a + cb_b * cb_b), 0.f);
    if (use_table) table_regs.store(cl.table);
    if constexpr (MODE == kTileScores) {
      if ((int)threadIdx.x * 4 < rep * kGroup) {
        const int e = threadIdx.x * 4, qh = e / kGroup, d = e % kGroup;
        f32x4 f;
        f.x = __uint_as_float(qreg.x << 16); f.y = __uint_as_float(qreg.x & 0xffff0000u);
        f.z = __uint_as_float(qreg.y << 16); f.w = __uint_as_float(qreg.y & 0xffff0000u);
        *reinterpret_cast<f32x4*>(q_lds + qh * kQueryLdsStride + (d / kValsPerLane) * kQueryLdsQuad + d % kValsPerLane) = f;
      }
    }
#pragma unroll
    for (int h = 0; h < kPasses; ++h) {
      constexpr int kParkRows = E::kParkRows, kBlocks = kParkRows / 32;        // row blocks per park; those of a wave lie S::WM apart
      const int ph = h % E::kParkPasses, first = h / E::kParkPasses * kBlocks;
      const int here = S::kRows - h * kPassRows < kPassRows ? S::kRows - h * kPassRows : kPassRows;   // rows of this pass
      if (ph == 0) {
        if (h > 0) __syncthreads();                             // the previous rows have been consumed
        static_assert(kBlocks % S::WM == 0, "blocks of a park");
        if (wave < kMulWaves) {
#pragma unroll
          for (int i = first / S::WM; i < S::MI && i * S::WM < first + kBlocks; ++i)
#pragma unroll
            for (int j = 0; j < S::NJ; ++j)
#pragma unroll
              for (int r = 0; r < 16; ++r)
                park[(S::block_row(i, wm) - first * 32 + (r >> 2) * 8 + fk * 4 + (r & 3)) * kLdP +
                     park_col<kVals>(S::block_col(j, wn) + frow)] = acc[i][j][r] + bv[j];
        }
      }
      if (h + 1 < kPasses) fetch(h + 1);
      if (ph == 0) __syncthreads();
      if (wave * kWaveRows < here) {                            // (a pass of fewer rows: the first waves)
        const int prow = ph * kPassRows + wave * kWaveRows + wrow, lrow = h * kPassRows + wave * kWaveRows + wrow;
        const bool active = lrow < n_rows;
        const int64_t rowc = m0 + (active ? lrow : n_rows - 1);
        const int64_t gid = rowc * H + head;
        const int64_t off = rowc * a.D + n0;
        float p[kVals], v[kVals];
        read_parked(park + prow * kLdP, q, p);
        if constexpr (kEnc) {
#pragma unroll
          for (int k = 0; k < kVals / 8; ++k) unpack_bf16x8(in[h & 1].x[k], &v[8 * k]);
          quantize_group<NCW, false, MB % 3 == 0 || S::MI >= 5 ? 4 : 8>(v, p, sf, q, cl.cb, use_table ? cl.table : nullptr, active, gid, a.codes, a.scales,
                              a.Xhat != nullptr);
        } else if constexpr (kWideGrid) {
          dequantize_across_heads<NCW>(wide[h & 1], in[h & 1].w.scale, head, q, p, sf, cl.cb, v);
        } else {
          dequantize_words<NCW>(in[h & 1].w, p, sf, q, cl.cb, v);
        }
        if (a.Xhat != nullptr && active) Storage<bf16_t>::store<false>(a.Xhat + off, q, v);
        if constexpr (MODE == kTileScores)
          score_row(v, q, head, H, a.q_heads, b, t0 + (active ? lrow : n_rows - 1), a.seq_len, active, a.q, a.score_scale,
                    a.scores, a.rope_cos, a.rope_sin, q_lds);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

template <int NCW, int MODE, int MB, bool WIDE, int SUMS>
__global__ __launch_bounds__(Tile<MB>::kThreads) __attribute__((amdgpu_waves_per_eu(Tile<MB>::kWaves / 4))) void fused_tile_kernel(const TileArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[TileEpilogue<MODE, MB>::kLdsBytes];
  fused_tile<NCW, MODE, MB, WIDE, SUMS>(a, (int)blockIdx.x, false, smem);
}
// Job `second` of the two at byte `at` of the kernel's arguments: read from where it was passed (an index into a copy would put them in
// scratch).
__device__ __forceinline__ TileArgs job_of_pair(int at, int second) {
  TileArgs a;
  __builtin_memcpy(&a, (const char*)__builtin_amdgcn_kernarg_segment_ptr() + at + second * (int)sizeof(TileArgs), sizeof(TileArgs));
  return a;
}
// Workgroup blockIdx.x of a launch for two jobs, the first `blocks` on job[0].
template <int NCW, int MODE, int MB, bool WIDE, int SUMS>
__device__ __forceinline__ void fused_tile_of_pair(int at, int blocks, unsigned char* smem) {
  const int second = (int)blockIdx.x >= blocks;
  const TileArgs a = job_of_pair(at, second);
  fused_tile<NCW, MODE, MB, WIDE, SUMS>(a, (int)blockIdx.x - (second ? blocks : 0), SUMS == kKeepSums && a.sums_hi != nullptr, smem);
}
// (a kernel of its own: picking the job puts another round of scalar loads ahead of everything, 0.4 us)
template <int NCW, int MODE, bool WIDE>
__global__ __launch_bounds__(Tile<1>::kThreads) __attribute__((amdgpu_waves_per_eu(Tile<1>::kWaves / 4))) void fused_tile_pair_kernel(const TilePair pair) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[TileEpilogue<MODE, 1>::kLdsBytes];
  fused_tile_of_pair<NCW, MODE, 1, WIDE, kKeepSums>(0, pair.blocks, smem);
}
// Two tensors that are encoded, or predicted (MODE)
template <int NCW, int MODE, int MB>
__global__ __launch_bounds__(Tile<MB>::kThreads) __attribute__((amdgpu_waves_per_eu(Tile<MB>::kWaves / 4))) void fused_tile_two_kernel(const TilePair pair) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[TileEpilogue<MODE, MB>::kLdsBytes];
  fused_tile_of_pair<NCW, MODE, MB, false, kNoSums>(0, pair.blocks, smem);
}
// The predictions of two tensors on tiles of different sizes
template <int MB0, int MB1, int WAVES = TwoTiles<MB0, MB1>::kWaves>
__global__ __launch_bounds__(WAVES * 64) __attribute__((amdgpu_waves_per_eu(WAVES / 4))) void predict_two_tiles_kernel(const TilePair pair) {
  constexpr int kLds0 = TileEpilogue<kTilePredict, MB0>::kLdsBytes, kLds1 = TileEpilogue<kTilePredict, MB1>::kLdsBytes;
  __shared__ __attribute__((aligned(16))) unsigned char smem[kLds0 > kLds1 ? kLds0 : kLds1];
  if ((int)blockIdx.x < pair.blocks) fused_tile<16, kTilePredict, MB0, false, kNoSums, WAVES>(job_of_pair(0, 0), (int)blockIdx.x, false, smem);
  else fused_tile<16, kTilePredict, MB1, false, kNoSums, WAVES>(job_of_pair(0, 1), (int)blockIdx.x - pair.blocks, false, smem);
}
// The pieces of a launch that workgroup `block` of those behind its tiles takes: one per kAttendThreads threads.
template <int THREADS>
__device__ __forceinline__ void attend_behind_tiles(AttendCacheParam& a, int block, unsigned char* smem) {
  constexpr int kPer = THREADS / kAttendThreads;
  const int part = __builtin_amdgcn_readfirstlane(threadIdx.x / kAttendThreads);
  const int items = (a.pieces.first[a.pieces.n_seq] - a.pieces.first[0]) * a.kv_heads, item = block * kPer + part;
  attend_piece<bf16_t>(a, item < items ? item : items - 1, (int)threadIdx.x % kAttendThreads, item < items,
                       reinterpret_cast<AttendLds*>(smem)[part]);
}
template <int NCW, int MB, bool WIDE>
__global__ __launch_bounds__(Tile<MB>::kThreads) __attribute__((amdgpu_waves_per_eu(Tile<MB>::kWaves / 4))) void fused_tile_attend_kernel(const TileAttend job) {
  constexpr int kTileBytes = TileEpilogue<kTileDecode, MB>::kLdsBytes, kAttendBytes = Tile<MB>::kThreads / kAttendThreads * (int)sizeof(AttendLds);
  __shared__ __attribute__((aligned(16))) unsigned char smem[kTileBytes > kAttendBytes ? kTileBytes : kAttendBytes];
  if ((int)blockIdx.x < job.tiles) {
    fused_tile_of_pair<NCW, kTileDecode, MB, WIDE, kNoSums>((int)offsetof(TileAttend, pair), job.pair.blocks, smem);
  } else {
    const char* const args = (const char*)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(TileAttend, attend);
    attend_behind_tiles<Tile<MB>::kThreads>(*(AttendCacheParam*)args, (int)blockIdx.x - job.tiles, smem);
  }
}

// rows per tile 32, 64, 96, 128, 192 or 320 (one translation unit each); tiles_per_seq is filled in
#define AQUAKV_TILE_LAUNCHER(ROWS) \
  hipError_t launch_tile_##ROWS(int mode, int n_codewords, bool wide, int n_seq, const TileArgs& a, hipStream_t stream)
AQUAKV_TILE_LAUNCHER(32);
AQUAKV_TILE_LAUNCHER(64);
AQUAKV_TILE_LAUNCHER(96);
AQUAKV_TILE_LAUNCHER(128);
AQUAKV_TILE_LAUNCHER(192);
AQUAKV_TILE_LAUNCHER(320);
// Two jobs of one mode and quantizer (TilePair), decode or encode, the second for sums if it has a place for them.
hipError_t launch_pair_32(int mode, int n_codewords, bool wide, const TileArgs& a, const TileArgs& b, hipStream_t stream);
// Decode of n = 1 or 2 jobs of one quantizer with pieces of attention behind their tiles (no pieces: those of no sequence).
#define AQUAKV_TILE_ATTEND_LAUNCHER(ROWS)                                                                                  \
  hipError_t launch_tile_attend_##ROWS(int n_codewords, bool wide, const TileArgs* jobs, int n, const AttendCacheArgs& attend, \
                                       hipStream_t stream)
AQUAKV_TILE_ATTEND_LAUNCHER(32);
AQUAKV_TILE_ATTEND_LAUNCHER(64);
AQUAKV_TILE_ATTEND_LAUNCHER(96);
AQUAKV_TILE_ATTEND_LAUNCHER(128);
AQUAKV_TILE_ATTEND_LAUNCHER(192);
// Encode or prediction of two jobs of one quantizer (tiles of 32 rows: prediction; launch_pair_32 encodes).
#define AQUAKV_TILE_TWO_LAUNCHER(ROWS) hipError_t launch_tile_two_##ROWS(int mode, int n_codewords, const TileArgs* jobs, hipStream_t stream)
AQUAKV_TILE_TWO_LAUNCHER(32);
AQUAKV_TILE_TWO_LAUNCHER(64);
AQUAKV_TILE_TWO_LAUNCHER(96);
AQUAKV_TILE_TWO_LAUNCHER(128);
AQUAKV_TILE_TWO_LAUNCHER(192);
// Predictions of two jobs on tiles of rows0 and rows1 rows: 32 and 96, 64 and 128, 64 and 192, 96 and 192 or 128 and 192.
hipError_t launch_predict_two_tiles(int rows0, int rows1, const TileArgs* jobs, hipStream_t stream);
// Tiles of 32 rows, encode or decode: a product that goes on from stored sums.
hipError_t launch_tile_rest(int mode, int n_codewords, bool wide, const TileArgs& a, hipStream_t stream);

#define AQUAKV_TILE_N(MODE, WIDE)                                  \
  do {                                                             \
    if (n_codewords == kRtn2) AQUAKV_TILE(kRtn2, MODE, WIDE);      \
    else if (n_codewords == kRtn4) AQUAKV_TILE(kRtn4, MODE, WIDE); \
    else if (n_codewords == 16) AQUAKV_TILE(16, MODE, WIDE);       \
    else if (n_codewords == 64) AQUAKV_TILE(64, MODE, WIDE);       \
    else AQUAKV_TILE(256, MODE, WIDE);                             \
  } while (0)

template <int MB>
hipError_t launch_tile(int mode, int n_codewords, bool wide, int n_seq, TileArgs a, hipStream_t stream) {
  using S = Tile<MB>;
  a.tiles_per_seq = (a.seq_len + S::kRows - 1) / S::kRows;
  const unsigned blocks = (unsigned)((int64_t)n_seq * a.tiles_per_seq * (a.D / kGroup));
  a.xcd = xcd_split((int64_t)n_seq * a.tiles_per_seq, a.D / kGroup, S::kRows);
#define AQUAKV_TILE(N, MODE, WIDE) fused_tile_kernel<N, MODE, MB, WIDE, kNoSums><<<blocks, S::kThreads, 0, stream>>>(a)
  if (mode == kTilePredict) AQUAKV_TILE(16, kTilePredict, false);
  else if (mode == kTileEncode) AQUAKV_TILE_N(kTileEncode, false);
  else if (mode == kTileDecode && wide) AQUAKV_TILE_N(kTileDecode, true);
  else if (mode == kTileDecode) AQUAKV_TILE_N(kTileDecode, false);
  else if (wide) AQUAKV_TILE_N(kTileScores, true);
  else AQUAKV_TILE_N(kTileScores, false);
#undef AQUAKV_TILE
  return hipGetLastError();
}

// fills in the jobs' tiles, returns how many there are
template <int MB0, int MB1 = MB0>
int pair_jobs(TilePair& pair, const TileArgs* jobs, int n) {
  int tiles = 0;
  for (int i = 0; i < 2; ++i) {
    const int rows = i == 0 ? Tile<MB0>::kRows : Tile<MB1>::kRows;
    TileArgs& job = pair.job[i];
    job = jobs[i < n ? i : 0];
    job.tiles_per_seq = (job.seq_len + rows - 1) / rows;
    job.xcd = xcd_split(job.tiles_per_seq, job.D / kGroup, rows);
    if (i < n) tiles += job.tiles_per_seq * (job.D / kGroup);
    if (i == 0) pair.blocks = tiles;
  }
  return tiles;
}

template <int MB>
hipError_t launch_tile_attend(int n_codewords, bool wide, const TileArgs* jobs, int n, const AttendCacheArgs& attend, hipStream_t stream) {
  using S = Tile<MB>;
  TileAttend args;
  args.tiles = pair_jobs<MB>(args.pair, jobs, n);
  args.attend = attend;
  const unsigned blocks = (unsigned)args.tiles + attend_workgroups(attend, S::kThreads);
#define AQUAKV_TILE(N, MODE, WIDE) fused_tile_attend_kernel<N, MB, WIDE><<<blocks, S::kThreads, 0, stream>>>(args)
  if (wide) AQUAKV_TILE_N(kTileDecode, true);
  else AQUAKV_TILE_N(kTileDecode, false);
#undef AQUAKV_TILE
  return hipGetLastError();
}

template <int MB>
hipError_t launch_tile_two(int mode, int n_codewords, const TileArgs* jobs, hipStream_t stream) {
  TilePair pair;
  const unsigned blocks = (unsigned)pair_jobs<MB>(pair, jobs, 2);
#define AQUAKV_TILE(N, MODE, WIDE) fused_tile_two_kernel<N, MODE, MB><<<blocks, Tile<MB>::kThreads, 0, stream>>>(pair)
  if (mode == kTilePredict) {
    AQUAKV_TILE(16, kTilePredict, false);
  } else if constexpr (MB > 1) {
    if (mode != kTileEncode) return hipErrorInvalidValue;
    AQUAKV_TILE_N(kTileEncode, false);
  } else {
    return hipErrorInvalidValue;
  }
#undef AQUAKV_TILE
  return hipGetLastError();
}

}  // namespace aquakv

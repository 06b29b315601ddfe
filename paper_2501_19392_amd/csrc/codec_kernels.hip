// Streaming kernels of the backbone quantizer (Sect. 2 "Vector Quantization" of
// the AQUA-KV paper, HIGGS-style): quantize (residual -> RHT -> group scale ->
// nearest grid point -> packed codes, plus the reconstruction), dequantize, and
// dequantize fused with grouped-query q.k scoring; plus the builder of the
// nearest-grid-point search table.  These are the stand-alone forms (prediction
// read from memory, or absent); the fused forms live in fused_kernels.hip.
//
// One head group (128 values) is held by eight lanes x 16 values (see device_utils.h; the scores kernel: a quad x 32);
// a 256-thread block covers 32 head groups = 4 tokens of 8 heads per pass.  WIDE = true selects
// rotation groups of 1024 = the whole token (the grouping of the paper's experiments, Sect. 4.1):
// the 64 lanes of a token = one wave then share three more butterfly stages and one scale.
#include "codec_core.h"
#include "kernels.h"

#include <numeric>

namespace aquakv {
namespace {

constexpr int kThreads = 256;
constexpr int kQuantizeVals = 16, kDequantizeVals = 16;      // values per lane
constexpr int kCodesVals = 32;                               // ... of the quantizer that writes codes only
constexpr int kGroupsPerBlock = kThreads / kLanesPerGroup;   // 64

// ------------------------------------------------------------------ quantize
// blockIdx.y: which of the one or two tensors of the launch (QuantizeIo in kernels.h; the keys and the values of a layer
// without predictors do not depend on each other, nor do the values of a layer and the keys of the next one, and together they fill
// the chip better).
//
// Without a prediction bound by vector issue: the vector pipes are busy in 0.94 of the cycles with 16 points (keys and values of 8192 tokens, groups
// of 1024, 29.9 us) and in 0.84 with 256 (37.4 us), where LDS is in 0.70, three fifths of that bank conflicts of the grid points' reads.  16 values per
// lane: 113 to 120 registers = four waves per SIMD (PRED false), 147 to 154 = three with a prediction.  With 32 values per lane it was three and
// two.  256 points: 36.6 us against 49.6; with predictions in memory, 4096 tokens, 16 points, predictor included, 88.5 against 114.7.
// With a prediction the vector pipes are busy in 0.73 (16 points) and 0.64 (256): 2.2 to 2.3 waves per SIMD on average do not cover the rest,
// start and drain of the few rounds and the look-ups' LDS latency (LDS busy in 0.34 and 0.50).  Predictions come from memory once (52.9
// MB fetched for a tensor of 8192 tokens, 50.3 of it rows and predictions): their second read is served by L2.  Smaller code for the
// crowded cells, which would let four or five waves in, changed nothing.
//
// CODES: no tensor of the launch wants its reconstruction (uniform backbone in bf16, without a prediction).  There is no search to
// request behind, so the next rows are requested ahead of this round's work, and no scattered store; what counts is the group's
// reductions and divisions per lane, hence 32 values.  Keys and values, 2 bits, groups across the heads, 35421 tokens: 27 us; 34 with
// 16 values requested behind the work, 33 ahead of it.  (With reconstructions 8192 tokens take 12.2 us on 16 values, 13.9 on 32.)
// Which launches: codes_pay.
template <typename T, int NCW, bool WIDE, bool PRED, bool CODES>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(PRED || CODES ? 3 : 4))) void quantize_kernel(
    const QuantizeIo io0, const QuantizeIo io1, const Prediction P0, const Prediction P1, const float* __restrict__ codebook,
    const uint32_t* __restrict__ table, int64_t n_groups, int H, bool fixed_head) {
  const T* const X = static_cast<const T*>(blockIdx.y ? io1.X : io0.X);
  T* const Xhat = CODES ? nullptr : static_cast<T*>(blockIdx.y ? io1.Xhat : io0.Xhat);
  const int8_t* const signs = blockIdx.y ? io1.signs : io0.signs;
  uint8_t* const codes = blockIdx.y ? io1.codes : io0.codes;
  uint16_t* const scales = blockIdx.y ? io1.scales : io0.scales;
  const Prediction P = {blockIdx.y ? P1.first : P0.first, blockIdx.y ? P1.second : P0.second, P0.stride, P0.split};
  __shared__ Lds lds;
  constexpr int N = CODES ? kCodesVals : kQuantizeVals, kLanes = kGroup / N, kGroups = kThreads / kLanes;       // lanes per group, groups per round
  const int l = WIDE ? token_pos<N>(threadIdx.x) : group_pos<N>(threadIdx.x), q = l & (kLanes - 1), slot = threadIdx.x / kLanes;
  // (a thread meets the same head in every round of the grid-stride loop: the signs are fetched once.  One that is behind the end repeats
  // the last group, with its signs: those of another head make a group that does not exist, whose search can take longer than any other's)
  float sf[N] = {};
  if constexpr (!is_rtn(NCW)) {
    const unsigned first = blockIdx.x * (unsigned)kGroups + slot;
    if (fixed_head) load_signs(signs, (int)((first < n_groups ? first : (unsigned)(n_groups - 1)) % (unsigned)H), q, sf);
  }
  // The rows (and the fp32 prediction) of the next round are requested behind this round's search: the inverse transform and the
  // stores hide some of their latency, the other waves of the SIMD the rest.  The prediction is read again for the reconstruction
  // instead of being held through the search (32 registers), but by the uniform backbone, which has registers to spare (4 bits, 35421
  // tokens with predictions 51 us, 59 when it read them twice).
  constexpr int kXQuads = N * sizeof(T) / 16, kPQuads = PRED ? N / 4 : 1;
  struct Rows { u32x4 x[kXQuads]; f32x4 p[kPQuads]; };
  // (groups across the heads: 8 heads, a lane meets the same one in every round and so one half of the predictions)
  const int p_col = (l / kLanes) * kGroup + q * N;
  const float* const p_half = p_col < P.split ? P.first + p_col : P.second + (p_col - P.split);
  const auto request_p = [&](int64_t gid, f32x4 (&r)[kPQuads]) {
    if constexpr (PRED) {
      const float* const src = WIDE ? p_half + (gid >> 3) * P.stride : P.first + (gid * kGroup + q * N);
#pragma unroll
      for (int k = 0; k < N / 4; ++k) r[k] = reinterpret_cast<const f32x4*>(src)[k];
    }
  };
  const auto unpack_p = [&](const f32x4 (&r)[kPQuads], float (&p)[N]) {
#pragma unroll
    for (int k = 0; k < N / 4; ++k) {
      const f32x4 a = PRED ? r[k % kPQuads] : f32x4{0.f, 0.f, 0.f, 0.f};
      p[4 * k] = a.x; p[4 * k + 1] = a.y; p[4 * k + 2] = a.z; p[4 * k + 3] = a.w;
    }
  };
  const auto request = [&](int64_t g0, Rows& r) {
    int64_t gid = g0 + slot;
    gid = gid < n_groups ? gid : n_groups - 1;
    const int64_t off = gid * kGroup + q * N;
    const u32x4* src = reinterpret_cast<const u32x4*>(X + off);
#pragma unroll
    for (int k = 0; k < kXQuads; ++k) r.x[k] = src[k];
    request_p(gid, r.p);
  };
  const int64_t stride = (int64_t)gridDim.x * kGroups;
  // The first rows are on their way while the grid and the table are staged, and all of the table's loads are out before the first is
  // stored: latencies one after the other are what a launch of few rounds is bound by (8192 x 1024 values at 4 bits: 36.6
  // -> 35.9 us of the call; the 17 layers of a cache of 2304 quantized tokens: 508 -> 503 us).
  Rows rows;
  if ((int64_t)blockIdx.x * kGroups < n_groups) request((int64_t)blockIdx.x * kGroups, rows);
  if constexpr (!is_rtn(NCW)) {
    static_assert(NCW <= kThreads, "one grid point per thread");
    TableRegs<kThreads> table_regs;
    if (table != nullptr) table_regs.request(table);
    load_codebook<NCW>(codebook, lds.cb);
    if (table != nullptr) table_regs.store(lds.table);
    __syncthreads();
  }
  for (int64_t g0 = (int64_t)blockIdx.x * kGroups; g0 < n_groups; g0 += stride) {
    int64_t gid = g0 + slot;
    const bool active = gid < n_groups;
    if (!active) gid = n_groups - 1;                      // keep every lane in the DPP exchanges

    float v[N], p[N];
    if constexpr (sizeof(T) == 2) {
#pragma unroll
      for (int k = 0; k < kXQuads; ++k) unpack_bf16x8(rows.x[k], &v[8 * k]);
    } else {
#pragma unroll
      for (int k = 0; k < N / 4; ++k) {
        v[4 * k] = __uint_as_float(rows.x[k].x); v[4 * k + 1] = __uint_as_float(rows.x[k].y);
        v[4 * k + 2] = __uint_as_float(rows.x[k].z); v[4 * k + 3] = __uint_as_float(rows.x[k].w);
      }
    }
    unpack_p(rows.p, p);
    if (CODES && g0 + stride < n_groups) request(g0 + stride, rows);
#pragma unroll
    for (int r = 0; r < N; ++r) v[r] -= p[r];
    if constexpr (!is_rtn(NCW)) {
      if (!fixed_head) load_signs(signs, (int)(gid % H), q, sf);     // (a 64-bit remainder: kept off the common path)
    }
    f32x4 again[kPQuads];
    quantize_residual<NCW, WIDE>(v, sf, l, lds.cb, table != nullptr ? lds.table : nullptr, active, gid, codes, scales,
                                 Xhat != nullptr, [&] {
      asm volatile("" ::: "memory");                      // (not the registers of the first read)
      if (!is_rtn(NCW) && Xhat != nullptr) request_p(gid, again);
      if (!CODES && g0 + stride < n_groups) request(g0 + stride, rows);
    });
    if (Xhat != nullptr) {
      if constexpr (!is_rtn(NCW)) unpack_p(again, p);
      if constexpr (WIDE && PRED) {                       // a wave's rows of P may lie under those it writes: all of it has been read
#pragma unroll
        for (int r = 0; r < N; ++r) asm volatile("" ::"v"(p[r]) : "memory");
      }
      finish_hat<NCW>(v, sf, p);
      if (active) Storage<T>::template store<false>(Xhat + gid * kGroup, q, v);
    }
  }
}

// ------------------------------------------------------------------ dequantize
// blockIdx.y: which of the one or two tensors of the launch (X unused)
// Bound by its stores, of which a lane with 16 values makes half as scattered ones as with 32 (16-byte pieces of 32 or of 64 bytes
// per lane: 5.6 against 3.3 TB/s), and by latency in few waves.  Keys and values without predictors, 16 points: 8192 tokens
// 15.1 -> 11.1 us, 131072 229 -> 171; 256 points, groups across the heads: 18.4 -> 14.7, 263 -> 198.
template <typename T, int NCW, bool WIDE>
__global__ __launch_bounds__(kThreads) void dequantize_kernel(const QuantizeIo io0, const QuantizeIo io1,
                                                              const float* __restrict__ P,
                                                              const float* __restrict__ codebook, int64_t n_groups, int H, bool fixed_head) {
  const uint8_t* __restrict__ const codes = blockIdx.y ? io1.codes : io0.codes;
  const uint16_t* __restrict__ const scales = blockIdx.y ? io1.scales : io0.scales;
  const int8_t* __restrict__ const signs = blockIdx.y ? io1.signs : io0.signs;
  T* __restrict__ const Xhat = static_cast<T*>(blockIdx.y ? io1.Xhat : io0.Xhat);
  __shared__ float4 cb[is_rtn(NCW) ? 1 : NCW];
  load_codebook<NCW>(codebook, cb);
  __syncthreads();
  constexpr int N = kDequantizeVals, kLanes = kGroup / N, kGroups = kThreads / kLanes;       // lanes per group, groups per round
  const int l = WIDE ? token_pos<N>(threadIdx.x) : group_pos<N>(threadIdx.x), q = l & (kLanes - 1), slot = threadIdx.x / kLanes;
  // (a thread meets the same head in every round of the grid-stride loop: the signs are fetched once)
  float sf[N] = {};
  if constexpr (!is_rtn(NCW)) {
    if (fixed_head) load_signs(signs, (int)((blockIdx.x * (unsigned)kGroups + slot) % (unsigned)H), q, sf);
  }
  // the code and scale words of the next round are requested before the current round is worked on
  const auto request = [&](int64_t g0) {
    int64_t gid = g0 + slot;
    gid = gid < n_groups ? gid : n_groups - 1;
    return request_words<NCW, WIDE, N>(codes, scales, gid, q);
  };
  const int64_t stride = (int64_t)gridDim.x * kGroups;
  CodeWords cur = {};
  if ((int64_t)blockIdx.x * kGroups < n_groups) cur = request((int64_t)blockIdx.x * kGroups);
  for (int64_t g0 = (int64_t)blockIdx.x * kGroups; g0 < n_groups; g0 += stride) {
    CodeWords nxt = {};
    if (g0 + stride < n_groups) nxt = request(g0 + stride);
    int64_t gid = g0 + slot;
    const bool active = gid < n_groups;
    if (!active) gid = n_groups - 1;
    const int64_t off = gid * kGroup + q * N;

    float p[N], z[N];
    if (P != nullptr) {
      load_f32(P + off, p);
    } else {
#pragma unroll
      for (int r = 0; r < N; ++r) p[r] = 0.f;
    }
    if constexpr (!is_rtn(NCW)) {
      if (!fixed_head) load_signs(signs, (int)(gid % H), q, sf);     // (a 64-bit remainder: kept off the common path)
    }
    dequantize_words<NCW, WIDE>(cur, p, sf, l, cb, z);
    if (active) Storage<T>::template store<false>(Xhat + gid * kGroup, q, z);
    cur = nxt;
  }
}

// ------------------------------------------------------------------ dequantize + q.k
// Group gid = row * H + head of the chunk; row = b * seq_len + t (global row = row0 + row).
template <typename T, int NCW, bool WIDE>
__global__ __launch_bounds__(kThreads) void attn_scores_kernel(
    const uint8_t* __restrict__ codes, const uint16_t* __restrict__ scales, const float* __restrict__ P,
    const int8_t* __restrict__ signs, const float* __restrict__ codebook, const T* __restrict__ qv_,
    float score_scale, float* __restrict__ scores, T* __restrict__ Khat_out, int64_t row0, int64_t n_groups,
    int seq_len, int H, int q_heads, const float* __restrict__ rope_cos, const float* __restrict__ rope_sin) {
  __shared__ float4 cb[is_rtn(NCW) ? 1 : NCW];
  load_codebook<NCW>(codebook, cb);
  __syncthreads();
  const int l = WIDE ? token_pos<32>(threadIdx.x) : (int)threadIdx.x & 3, q = l & 3;
  // A thread meets the same head in every round of the grid-stride loop when the groups of a block are a multiple of H (they
  // are for powers of two up to 64): the signs are then fetched once.
  float sf[32] = {};
  const bool fixed_head = kGroupsPerBlock % H == 0;
  if constexpr (!is_rtn(NCW)) {
    if (fixed_head) load_signs(signs, (int)((blockIdx.x * (unsigned)kGroupsPerBlock + (threadIdx.x >> 2)) % (unsigned)H), q, sf);
  }
  const int rep = q_heads / H;
  const auto request = [&](int64_t g0) {
    int64_t gid = g0 + (threadIdx.x >> 2);
    gid = gid < n_groups ? gid : n_groups - 1;
    return request_words<NCW, WIDE>(codes, scales, gid, q);
  };
  const int64_t stride = (int64_t)gridDim.x * kGroupsPerBlock;
  CodeWords cur = {};
  if ((int64_t)blockIdx.x * kGroupsPerBlock < n_groups) cur = request((int64_t)blockIdx.x * kGroupsPerBlock);
  for (int64_t g0 = (int64_t)blockIdx.x * kGroupsPerBlock; g0 < n_groups; g0 += stride) {
    CodeWords nxt = {};
    if (g0 + stride < n_groups) nxt = request(g0 + stride);
    int64_t gid = g0 + (threadIdx.x >> 2);
    const bool active = gid < n_groups;
    if (!active) gid = n_groups - 1;
    const int head = (int)(gid % H);
    const int64_t row = row0 + gid / H;
    const int64_t b = row / seq_len;
    const int64_t t = row % seq_len;
    const int64_t off = gid * kGroup + q * kValsPerLane;

    float p[32], z[32];
    if (P != nullptr) {
      load_f32(P + off, p);
    } else {
#pragma unroll
      for (int r = 0; r < 32; ++r) p[r] = 0.f;
    }
    if constexpr (!is_rtn(NCW)) {
      if (!fixed_head) load_signs(signs, (int)(gid % H), q, sf);     // (a 64-bit remainder: kept off the common path)
    }
    dequantize_words<NCW, WIDE>(cur, p, sf, l, cb, z);
    cur = nxt;
    if (Khat_out != nullptr && active) Storage<T>::template store<WIDE>(Khat_out + gid * kGroup, q, z);
#pragma unroll
    for (int r = 0; r < 32; ++r) z[r] = Storage<T>::round(z[r]);      // score the stored keys
    if (rope_cos != nullptr) rope128(z, q, rope_cos + t * (kGroup / 2), rope_sin + t * (kGroup / 2));   // cached before RoPE

    for (int r = 0; r < rep; ++r) {
      const int qh = head * rep + r;
      float qv[32];
      Storage<T>::load(qv_ + ((int64_t)b * q_heads + qh) * kGroup + q * kValsPerLane, qv);
      float acc = 0.f;
#pragma unroll
      for (int i = 0; i < 32; ++i) acc = __fmaf_rn(qv[i], z[i], acc);
      acc = quad_sum(acc);
      if (active && q == 0) scores[((int64_t)b * q_heads + qh) * seq_len + t] = acc * score_scale;
    }
  }
}

// ------------------------------------------------------------------ search table builder
// Grid point j is dropped from a cell only if some single other point i is closer by more than `eps` everywhere in
// the enlarged cell.  d_j(y) - d_i(y) = -2 y.(C_j - C_i) + |C_j|^2 - |C_i|^2 is linear in y, so its minimum over the
// rectangle sits at a corner; border cells reach out to +-1e30 (a clamped scale lets |y| grow without bound).
// The list is a superset of the points that can win anywhere in the cell, also under the kernels' fp32 rounding.
// Returns the number of candidates; the first kOvfCand of them (indices, ascending) go to cand[].
__device__ int cell_candidates(const float* __restrict__ codebook, int n, int cell, int (&cand)[kOvfCand]) {
  const int cx = cell % kCells, cy = cell / kCells;
  const double far = 1e30;
  const double delta = 1e-4, eps = 1e-3;
  const double R = cell_half_range(n);
  const double h = 2.0 * R / kCells;
  double x0 = cx == 0 ? -far : -R + cx * h, x1 = cx == kCells - 1 ? far : -R + (cx + 1) * h;
  double y0 = cy == 0 ? -far : -R + cy * h, y1 = cy == kCells - 1 ? far : -R + (cy + 1) * h;
  x0 -= delta; y0 -= delta; x1 += delta; y1 += delta;
  const double cxs[4] = {x0, x1, x0, x1}, cys[4] = {y0, y0, y1, y1};
  int count = 0;
  for (int j = 0; j < n; ++j) {
    const double aj = codebook[2 * j], bj = codebook[2 * j + 1];
    bool dominated = false;
    for (int i = 0; i < n && !dominated; ++i) {
      if (i == j) continue;
      const double ai = codebook[2 * i], bi = codebook[2 * i + 1];
      const double gx = -2.0 * (aj - ai), gy = -2.0 * (bj - bi);
      const double c0 = (aj * aj + bj * bj) - (ai * ai + bi * bi);
      double mn = 1e300;
      for (int k = 0; k < 4; ++k) mn = fmin(mn, gx * cxs[k] + gy * cys[k] + c0);
      dominated = mn > eps;
    }
    if (!dominated) {
#pragma unroll
      for (int k = 0; k < kOvfCand; ++k)
        if (k == count) cand[k] = j;
      ++count;
    }
  }
  return count;
}

// candidates -> `bytes` slot bytes, ascending, the last one repeated (little-endian into 32-bit words)
__device__ void pack_candidates(const int (&cand)[kOvfCand], int count, int shift, int bytes, uint32_t (&w)[2]) {
  w[0] = w[1] = 0;
#pragma unroll
  for (int k = 0; k < kOvfCand; ++k) {
    int c = 0;
#pragma unroll
    for (int t = 0; t < kOvfCand; ++t)
      if (t == (k < count ? k : count - 1)) c = cand[t];
    if (k < bytes) w[k >> 2] |= (uint32_t)(c << shift) << (8 * (k & 3));
  }
}

// First pass, one thread per cell: the ordinary entries; cells that need an overflow list of their own are left marked
// "full search".  With 256 points the cells that list nothing but point 255 name the shared list 0.
__global__ void build_table_kernel(const float* __restrict__ codebook, int n, uint32_t* __restrict__ table) {
  const int cell = blockIdx.x * blockDim.x + threadIdx.x;
  if (cell >= kCellWords) return;
  int cand[kOvfCand];
  const int count = cell_candidates(codebook, n, cell, cand);
  uint32_t w[2];
  pack_candidates(cand, count < 4 ? count : 4, slot_shift(n), 4, w);
  const bool ordinary = count <= (n == 16 ? 3 : 4) && w[0] < crowded_threshold(n);
  const bool only_last = n == 256 && count == 1 && cand[0] == n - 1;
  table[cell] = ordinary ? w[0] : crowded_entry(n, only_last ? 0u : slot_top(n));
}

// Second pass, one workgroup: the marked cells get overflow lists in cell order (a fixed table for a given grid).  A cell
// with more than kOvfCand candidates, or one that finds no list left, stays "full search".
__global__ __launch_bounds__(1024) void build_overflow_kernel(const float* __restrict__ codebook, int n,
                                                              uint32_t* __restrict__ table) {
  __shared__ int offs[1024];
  constexpr int kPer = kCellWords / 1024;
  const uint32_t marked = crowded_entry(n, slot_top(n));
  int mine = 0;
  for (int k = 0; k < kPer; ++k) mine += table[threadIdx.x * kPer + k] == marked;
  offs[threadIdx.x] = mine;
  __syncthreads();
  for (int d = 1; d < 1024; d <<= 1) {                    // inclusive scan
    const int add = (int)threadIdx.x >= d ? offs[threadIdx.x - d] : 0;
    __syncthreads();
    offs[threadIdx.x] += add;
    __syncthreads();
  }
  const int first = n == 256 ? 1 : 0;                     // list 0 of the 256-point grid: point 255 alone
  int list = first + offs[threadIdx.x] - mine;            // lists before this thread's cells
  // unused lists name point 0; the shared list names the last point in every byte
  for (int k = threadIdx.x; k < 2 * kOvfLists; k += 1024) table[kCellWords + k] = (first && k < 2) ? 0xFFFFFFFFu : 0u;
  __syncthreads();
  for (int k = 0; k < kPer; ++k) {
    const int cell = threadIdx.x * kPer + k;
    if (table[cell] != marked) continue;
    int cand[kOvfCand];
    const int count = cell_candidates(codebook, n, cell, cand);
    if (count <= kOvfCand && list < ovf_capacity(n)) {
      uint32_t w[2];
      pack_candidates(cand, count, slot_shift(n), kOvfCand, w);
      table[kCellWords + 2 * list] = w[0];
      table[kCellWords + 2 * list + 1] = w[1];
      table[cell] = crowded_entry(n, (uint32_t)list << slot_shift(n));
    }
    ++list;
  }
}

// Workgroups per CU (256 CUs), the kernels grid-stride.  The quantizer stages 21 KiB of grid and cell table per workgroup,
// more than the 8 KiB of rows of one round: with the resident number of workgroups the staging is paid once and
// the request of the next round's rows has a next round to run ahead of (more than those where it evens out the CUs: rounds_for).  The inverse stages 256 B to 4 KiB; keys and values of
// 131072 tokens, 16 points: 171 us with four workgroups per CU, 178 with six or eight (of 8192 tokens 11.1 with any of them).
// Below that number the rounds are shared out evenly.
//
// 32 values per lane for codes alone (n_groups head groups in all tensors).  Groups across the heads: as soon as 16 values would take more
// than a few waves per SIMD, two more reductions per lane then cost more than the waves cover (tokens of one tensor, 2 bits, us, 16 / 32
// values: 1000 2.6 / 2.9, 2000 3.0 / 2.9, 6000 4.7 / 4.1, 28000 15.5 / 14.2).  Groups of one head need few reductions: over many rounds
// only (keys and values: 1000 2.9 / 3.0, 10000 10.8 / 11.3, 16384 15.6 / 15.3, 20000 18.4 / 18.5, 21071 19.5 / 17.8, 131072 104 / 93).
inline bool codes_pay(int64_t n_groups, bool wide) { return n_groups >= (wide ? 16384 : 262144); }
constexpr int kQuantizeWgPerCu = 3, kQuantizePlainWgPerCu = 4, kCodesWgPerCu = 3;     // with a prediction, without, codes only
constexpr int kQuantizeStart = 2;
constexpr int kDequantizeWgPerCu = 4;
inline int64_t blocks_of_rounds(int64_t blocks, int64_t cap) {
  const int64_t rounds = (blocks + cap - 1) / cap;
  return (blocks + rounds - 1) / rounds;
}
// ... such that a thread meets the same head in every round, if the workgroups for that are resident.  4096 tokens of 64 heads: inverse
// 17.1 us (18.8 with a 64-bit remainder and the signs fetched in every round), quantizer with predictions, 256 points, 70.8 (73.2),
// which is what 32768 tokens of 8 heads take.
struct Rounds { unsigned blocks; bool fixed_head; };
// start != 0 (quarters of a round that a workgroup's start costs): more workgroups than are resident, of fewer rounds each, where the CUs then
// have fewer rounds to do.  With the resident number a CU does as many rounds as its busiest place: of 6500 tokens x 2 tensors some CUs have three
// workgroups of 4 rounds and others four, 36.1 us (256 points); 1626 workgroups of one or two rounds, dealt out as places get free, 31.7.
// 9000 tokens 45.5 / 41.2; 10007 tokens with predictions 27.6 / 26 a tensor.  Equal shares (8192 tokens) stay as they are.
inline Rounds rounds_for(int64_t n_groups, int groups_per_block, int H, int per_cu, int tensors, int start = 0) {
  const int64_t need = (n_groups + groups_per_block - 1) / groups_per_block, resident = 256 * per_cu / tensors;
  int64_t blocks = blocks_of_rounds(need, resident);
  if (blocks == need) return {(unsigned)blocks, true};
  const int64_t step = H / std::gcd(H, groups_per_block);       // blocks whose groups are a multiple of H
  if (start != 0) {
    const auto cost = [&](int64_t b) {
      return (b * tensors + 255) / 256 * (4 * ((need + b - 1) / b) + start);
    };
    int64_t best = blocks;
    for (int64_t r = 1; r * resident < need; ++r) {
      const int64_t b = ((need + r - 1) / r + step - 1) / step * step;
      if (cost(b) < cost(best)) best = b;
    }
    if (best != blocks) return {(unsigned)best, true};
  }
  const int64_t whole = (blocks + step - 1) / step * step;
  return whole <= resident ? Rounds{(unsigned)whole, true} : Rounds{(unsigned)blocks, false};
}

}  // namespace

#define AQUAKV_DISPATCH_GRID(NCW, CALL)                                                 \
  do {                                                                                  \
    if ((NCW) == 16) { constexpr int N = 16; CALL; }                                    \
    else if ((NCW) == 64) { constexpr int N = 64; CALL; }                               \
    else { constexpr int N = 256; CALL; }                                               \
  } while (0)
#define AQUAKV_DISPATCH_N(NCW, CALL)                                                    \
  do {                                                                                  \
    if ((NCW) == kRtn2) { constexpr int N = kRtn2; CALL; }                              \
    else if ((NCW) == kRtn4) { constexpr int N = kRtn4; CALL; }                         \
    else AQUAKV_DISPATCH_GRID(NCW, CALL);                                               \
  } while (0)
// binds T (storage type), N (quantizer id: grid size, or kRtn2 / kRtn4) and W (groups of 1024 = the whole token)
// as compile-time names for CALL
#define AQUAKV_DISPATCH(DT, NCW, WIDE_, CALL)                                           \
  do {                                                                                  \
    if ((DT) == kBF16) {                                                                \
      typedef bf16_t T;                                                                 \
      if (WIDE_) { constexpr bool W = true; AQUAKV_DISPATCH_N(NCW, CALL); }             \
      else { constexpr bool W = false; AQUAKV_DISPATCH_N(NCW, CALL); }                  \
    } else {                                                                            \
      typedef float T;                                                                  \
      if (WIDE_) { constexpr bool W = true; AQUAKV_DISPATCH_N(NCW, CALL); }             \
      else { constexpr bool W = false; AQUAKV_DISPATCH_N(NCW, CALL); }                  \
    }                                                                                   \
  } while (0)

hipError_t launch_build_search_table(const float* codebook, int n_codewords, void* table, hipStream_t stream) {
  build_table_kernel<<<kCellWords / 64, 64, 0, stream>>>(codebook, n_codewords, static_cast<uint32_t*>(table));
  build_overflow_kernel<<<1, 1024, 0, stream>>>(codebook, n_codewords, static_cast<uint32_t*>(table));
  return hipGetLastError();
}

hipError_t launch_quantize(int dtype, int n_codewords, const QuantizeIo* io, int tensors, const Prediction* P,
                           const float* codebook, const void* table, int64_t T_, int H, bool wide, hipStream_t stream) {
  const int64_t n_groups = T_ * H;
  if (n_groups == 0) return hipSuccess;
  for (int i = 0; i < tensors && P != nullptr; ++i) {
    if (P[i].stride != P[0].stride || P[i].split != P[0].split) return hipErrorInvalidValue;
    if (!wide && P[i].second != P[i].first + P[i].split) return hipErrorInvalidValue;             // (read as contiguous)
  }
  const QuantizeIo& other = io[tensors - 1];
  const uint32_t* tab = static_cast<const uint32_t*>(table);
  const bool codes_only = is_rtn(n_codewords) && dtype == kBF16 && P == nullptr && io[0].Xhat == nullptr && other.Xhat == nullptr &&
                          codes_pay(n_groups * tensors, wide);
  const int per_cu = P != nullptr ? kQuantizeWgPerCu : codes_only ? kCodesWgPerCu : kQuantizePlainWgPerCu;
  const Rounds r = rounds_for(n_groups, kThreads * (codes_only ? kCodesVals : kQuantizeVals) / kGroup, H, per_cu, tensors, kQuantizeStart);
  const dim3 grid(r.blocks, (unsigned)tensors);
  const Prediction p0 = P != nullptr ? P[0] : Prediction{}, p1 = P != nullptr ? P[tensors - 1] : Prediction{};
#define AQUAKV_QUANTIZE(T, N, W, PRED, CODES) \
  quantize_kernel<T, N, W, PRED, CODES><<<grid, kThreads, 0, stream>>>(io[0], other, p0, p1, codebook, tab, n_groups, H, r.fixed_head)
  if (codes_only) {
    if (n_codewords == kRtn2 && wide) AQUAKV_QUANTIZE(bf16_t, kRtn2, true, false, true);
    else if (n_codewords == kRtn2) AQUAKV_QUANTIZE(bf16_t, kRtn2, false, false, true);
    else if (wide) AQUAKV_QUANTIZE(bf16_t, kRtn4, true, false, true);
    else AQUAKV_QUANTIZE(bf16_t, kRtn4, false, false, true);
  } else if (P != nullptr) {
    AQUAKV_DISPATCH(dtype, n_codewords, wide, (AQUAKV_QUANTIZE(T, N, W, true, false)));
  } else {
    AQUAKV_DISPATCH(dtype, n_codewords, wide, (AQUAKV_QUANTIZE(T, N, W, false, false)));
  }
#undef AQUAKV_QUANTIZE
  return hipGetLastError();
}

hipError_t launch_dequantize(int dtype, int n_codewords, const QuantizeIo* io, int tensors, const float* P,
                             const float* codebook, int64_t T_, int H, bool wide, hipStream_t stream) {
  const int64_t n_groups = T_ * H;
  if (n_groups == 0) return hipSuccess;
  if (tensors != 1 && P != nullptr) return hipErrorInvalidValue;
  const Rounds r = rounds_for(n_groups, kThreads * kDequantizeVals / kGroup, H, kDequantizeWgPerCu, tensors);
  const dim3 grid(r.blocks, (unsigned)tensors);
  AQUAKV_DISPATCH(dtype, n_codewords, wide, (dequantize_kernel<T, N, W><<<grid, kThreads, 0, stream>>>(
                                                io[0], io[tensors - 1], P, codebook, n_groups, H, r.fixed_head)));
  return hipGetLastError();
}

hipError_t launch_attn_scores(int dtype, int n_codewords, const uint8_t* codes, const uint16_t* scales, const float* P,
                              const int8_t* signs, const float* codebook, const void* q, float score_scale,
                              float* scores, void* Khat_out, int64_t row0, int64_t rows, int seq_len, int H,
                              int q_heads, const float* rope_cos, const float* rope_sin, bool wide, hipStream_t stream) {
  const int64_t n_groups = rows * H;
  if (n_groups == 0) return hipSuccess;
  const unsigned blocks = (unsigned)blocks_of_rounds((n_groups + kGroupsPerBlock - 1) / kGroupsPerBlock, 256 * kDequantizeWgPerCu);
  AQUAKV_DISPATCH(dtype, n_codewords, wide,
                  (attn_scores_kernel<T, N, W><<<blocks, kThreads, 0, stream>>>(
                      codes, scales, P, signs, codebook, static_cast<const T*>(q), score_scale, scores,
                      static_cast<T*>(Khat_out), row0, n_groups, seq_len, H, q_heads, rope_cos, rope_sin)));
  return hipGetLastError();
}

}  // namespace aquakv

// One piece of the attention over a cache (attend_cache.hip) as a device function: the body of attend_cache_kernel, and work for the
// CUs that the recovery of the next layer leaves idle (fused_tile.h, fused_kernels.hip).
#pragma once
#include "device_utils.h"
#include "kernels.h"

namespace aquakv {

constexpr int kAttendThreads = 256;                   // of a workgroup work on a piece
constexpr int kAttendMaxRep = 8;                      // query heads worked on at a time
struct AttendLds {
  float q[kAttendMaxRep][kGroup];
  float sums[4][kAttendMaxRep][kGroup];
  float wave_stats[4][kAttendMaxRep][2];
};

// workgroups of `threads` for the pieces of a launch
inline unsigned attend_workgroups(const AttendCacheArgs& a, int threads) {
  const int64_t items = (int64_t)(a.pieces.first[a.pieces.n_seq] - a.pieces.first[0]) * a.kv_heads, per = threads / kAttendThreads;
  return (unsigned)((items + per - 1) / per);
}

namespace attend {

constexpr int kPasses = kAttendPiece / 16;            // 16 lanes per token, 16 tokens per pass of the workgroup
static_assert(kPasses == 4, "a quad of lanes shares the exponentials of its four tokens");
constexpr int kMaxRep = kAttendMaxRep;

template <int C> __device__ __forceinline__ float dpp(float x) {      // x of the lane that DPP control C names
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), C, 0xf, 0xf, true));
}
// The sums over the 16 lanes of a token for the token of each pass, lane i of a quad getting that of pass i: two lanes exchange what
// each sums for the other, so the work halves where a sum of all four in every lane repeats it.
__device__ __forceinline__ float sum16(const float (&d)[kPasses], int lane) {
  const bool odd = lane & 1, upper = lane & 2;
  const float a = (odd ? d[1] : d[0]) + dpp<0xb1>(odd ? d[0] : d[1]);          // quad_perm 1 0 3 2
  const float b = (odd ? d[3] : d[2]) + dpp<0xb1>(odd ? d[2] : d[3]);
  float x = (upper ? b : a) + dpp<0x4e>(upper ? a : b);                        // quad_perm 2 3 0 1
  x = x + dpp<0x128>(x);                              // row_ror:8; in this order all quads of the token end with the same bits
  return x + dpp<0x124>(x);                           // row_ror:4
}

// Reductions over the four groups of 16 lanes of a wave (a wave's tokens of one pass).  The gfx950 lane swaps exchange halves
// between two registers, v_permlane32_swap the upper 32 lanes of the first with the lower 32 of the second, v_permlane16_swap
// the odd groups of the first with the even ones of the second: adding the pair reduces two values at once, and they cost no
// trip through LDS as shuffles do.
__device__ __forceinline__ float fold32(float x, float y) {      // lanes < 32: x over both halves, lanes >= 32: y
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float fold16(float x, float y) {      // even groups: x over the pair of groups, odd groups: y
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float max_quad(float x) {
  x = fmaxf(x, dpp<0xb1>(x));                          // quad_perm 1 0 3 2
  return fmaxf(x, dpp<0x4e>(x));                       // quad_perm 2 3 0 1
}
__device__ __forceinline__ float max_groups(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Lane l of a token holds coordinates 4 l ... and 64 + 4 l ... of the key (pairs of the rotary embedding) and 8 l ... of the value.
template <typename T> struct Row;
template <> struct Row<bf16_t> {
  u32x2 lo, hi;
  u32x4 v;
  __device__ __forceinline__ void load(const bf16_t* k, const bf16_t* val, int l) {
    lo = *reinterpret_cast<const u32x2*>(k + 4 * l);
    hi = *reinterpret_cast<const u32x2*>(k + 64 + 4 * l);
    v = *reinterpret_cast<const u32x4*>(val + 8 * l);
  }
  static __device__ __forceinline__ void unpack4(const u32x2& u, float (&f)[8], int at) {
    f[at] = __uint_as_float(u.x << 16); f[at + 1] = __uint_as_float(u.x & 0xffff0000u);
    f[at + 2] = __uint_as_float(u.y << 16); f[at + 3] = __uint_as_float(u.y & 0xffff0000u);
  }
  __device__ __forceinline__ void key(float (&f)[8]) const { unpack4(lo, f, 0); unpack4(hi, f, 4); }
  __device__ __forceinline__ void value(float (&f)[8]) const { unpack_bf16x8(v, f); }
  __device__ __forceinline__ void no_value() { v = u32x4{0, 0, 0, 0}; }
};
template <> struct Row<float> {
  f32x4 lo, hi, v0, v1;
  __device__ __forceinline__ void load(const float* k, const float* val, int l) {
    lo = *reinterpret_cast<const f32x4*>(k + 4 * l);
    hi = *reinterpret_cast<const f32x4*>(k + 64 + 4 * l);
    v0 = *reinterpret_cast<const f32x4*>(val + 8 * l);
    v1 = *reinterpret_cast<const f32x4*>(val + 8 * l + 4);
  }
  static __device__ __forceinline__ void put4(const f32x4& u, float (&f)[8], int at) {
    f[at] = u.x; f[at + 1] = u.y; f[at + 2] = u.z; f[at + 3] = u.w;
  }
  __device__ __forceinline__ void key(float (&f)[8]) const { put4(lo, f, 0); put4(hi, f, 4); }
  __device__ __forceinline__ void value(float (&f)[8]) const { put4(v0, f, 0); put4(v1, f, 4); }
  __device__ __forceinline__ void no_value() { v0 = v1 = f32x4{0.f, 0.f, 0.f, 0.f}; }
};

}  // namespace attend

// item = piece * kv heads + head, of the launch's pieces; tid: the thread among the kAttendThreads that work on it.  `active`: the item
// is there (its results are stored); the barriers are met either way.  All rows of the piece are requested at once; thread (ts = tid / 16, l = tid % 16) owns
// tokens ts, ts + 16, ... of it.  Every wave takes the soft-max of its own tokens, so the waves meet once, to merge.
// part[piece, q_heads, 128]: sums with weights exp(score - maximum); stats[piece, q_heads, 2]: maximum and sum of the weights.
// Bound by the instructions per query head and the workgroups per CU, hence the scores shared out in a quad, the lane swaps, the short
// way to the addresses of compressed tokens only, and rows that are unpacked ahead of the loop (100 registers: four workgroups per
// CU, where 166 left room for three).  8 kv heads, in a trace: four sequences of up to 1800 tokens, 32 query heads, rotary embedding
// 11.3 us (13.1 with all four scores in every lane and 166 registers), 8000 tokens of 24 query heads 10.7 (13.7), 8 x 1000 tokens
// of 64 query heads 17.5 (20.6).  200 tokens: 6.7 us, which is launch and memory latency.
// `a`: the arguments where the launch put them, found with __builtin_amdgcn_kernarg_segment_ptr (a reference to a kernel's parameter would
// put a copy into scratch, because its arrays are indexed).
typedef const __attribute__((address_space(4))) AttendCacheArgs AttendCacheParam;
template <typename T>
__device__ __forceinline__ void attend_piece(AttendCacheParam& a, int item, int tid, bool active, AttendLds& lds) {
  using namespace attend;
  const int head = item % a.kv_heads, piece = a.pieces.first[0] + item / a.kv_heads;
  int b = 0;
  for (int step = kAttendSeqs / 2; step > 0; step >>= 1)
    if (b + step < a.pieces.n_seq && a.pieces.first[b + step] <= piece) b += step;
  const int rep = a.q_heads / a.kv_heads;
  const int lane = tid & 63, wave = tid >> 6;
  const int ts = tid >> 4, l = tid & 15;
  const int t0 = (piece - a.pieces.first[b]) * kAttendPiece;
  const int ns = a.n_sink[b], nc = a.n_compressed[b], n = a.n_tokens[b];
  const int64_t row_elems = (int64_t)a.kv_heads * kGroup;
  const int64_t seq = a.seq0 + b;

  Row<T> rows[kPasses];
  if (t0 >= ns && t0 + kAttendPiece <= ns + nc) {      // compressed tokens only: rows one after the other
    const int64_t off = (a.compressed_row[b] + t0 - ns) * row_elems + head * kGroup;
    const T *kb = static_cast<const T*>(a.compressed_k) + off, *vb = static_cast<const T*>(a.compressed_v) + off;
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
      const uint32_t at = (uint32_t)(p * 16 + ts) * (uint32_t)row_elems;
      rows[p].load(kb + at, vb + at, l);
    }
  } else {
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
      int t = t0 + p * 16 + ts;
      t = t < n ? t : n - 1;                           // beyond the end: weight 0 below
      const void *kb = a.sink_k, *vb = a.sink_v;
      int64_t row = seq * a.sink_rows + t;
      if (t >= ns) { kb = a.compressed_k; vb = a.compressed_v; row = a.compressed_row[b] + t - ns; }
      if (t >= ns + nc) { kb = a.recent_k; vb = a.recent_v; row = seq * a.recent_rows + t - ns - nc; }
      const int64_t off = row * row_elems + head * kGroup;
      rows[p].load(static_cast<const T*>(kb) + off, static_cast<const T*>(vb) + off, l);
    }
  }
  f32x4 cs[kPasses], sn[kPasses];
  if (a.rope_cos != nullptr) {
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
      int t = t0 + p * 16 + ts;
      t = t < n ? t : n - 1;
      cs[p] = *reinterpret_cast<const f32x4*>(a.rope_cos + (int64_t)t * 64 + 4 * l);
      sn[p] = *reinterpret_cast<const f32x4*>(a.rope_sin + (int64_t)t * 64 + 4 * l);
    }
  }
  if (t0 + kAttendPiece > n) {                         // beyond the end: the last token's values again, and 0 x infinity is no 0
#pragma unroll
    for (int p = 0; p < kPasses; ++p)
      if (t0 + p * 16 + ts >= n) rows[p].no_value();
  }
  const auto stage_queries = [&](int r0) {
    const int nr = rep - r0 < kMaxRep ? rep - r0 : kMaxRep;
    const T* qp = static_cast<const T*>(a.q) + (seq * a.q_heads + head * rep + r0) * kGroup;
    for (int e = tid; e < nr * kGroup; e += kAttendThreads) lds.q[e / kGroup][e % kGroup] = static_cast<float>(qp[e]);
  };
  stage_queries(0);
  float k[kPasses][8], v[kPasses][8];
#pragma unroll
  for (int p = 0; p < kPasses; ++p) {
    rows[p].key(k[p]);
    rows[p].value(v[p]);
    if (a.rope_cos != nullptr) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float x0 = k[p][i], x1 = k[p][4 + i];
        k[p][i] = __fmaf_rn(x0, cs[p][i], -(x1 * sn[p][i]));
        k[p][4 + i] = __fmaf_rn(x1, cs[p][i], x0 * sn[p][i]);
      }
    }
  }
  for (int r0 = 0; r0 < rep; r0 += kMaxRep) {
    const int nr = rep - r0 < kMaxRep ? rep - r0 : kMaxRep;
    const int qh0 = head * rep + r0;
    __syncthreads();                                   // the queries are there, the sums of the heads before them read
#pragma unroll 1
    for (int r = 0; r < nr; ++r) {
      const f32x4 q0 = *reinterpret_cast<const f32x4*>(&lds.q[r][4 * l]), q1 = *reinterpret_cast<const f32x4*>(&lds.q[r][64 + 4 * l]);
      const float q[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
      float d[kPasses] = {};
#pragma unroll
      for (int p = 0; p < kPasses; ++p)
#pragma unroll
        for (int i = 0; i < 8; ++i) d[p] = __fmaf_rn(q[i], k[p][i], d[p]);
      // each lane of a quad takes the exponential of one of the token's four scores, and the quad passes them round
      float mine = sum16(d, lane) * a.scale;
      if (t0 + (lane & 3) * 16 + ts >= n) mine = -INFINITY;
      const float m = max_groups(max_quad(mine));
      const float shift = m == -INFINITY ? 0.f : m;    // a wave without tokens
      const float weight = expf(mine - shift);
      float sum = quad_sum(weight), acc[8] = {};
#pragma unroll
      for (int p = 0; p < kPasses; ++p) {
        const float e = p == 0 ? dpp<0x00>(weight) : p == 1 ? dpp<0x55>(weight) : p == 2 ? dpp<0xaa>(weight) : dpp<0xff>(weight);
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = __fmaf_rn(e, v[p][i], acc[i]);
      }
      sum = fold32(sum, sum);
      sum = fold16(sum, sum);
      // lane group g ends with coordinates 4 (g / 2) + 2 (g % 2) ... of the lane's eight
      float f[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) f[i] = fold32(acc[i], acc[4 + i]);
      f32x2 o;
      o.x = fold16(f[0], f[2]);
      o.y = fold16(f[1], f[3]);
      *reinterpret_cast<f32x2*>(&lds.sums[wave][r][8 * l + 2 * (lane >> 4)]) = o;
      if (lane == 0) { lds.wave_stats[wave][r][0] = m; lds.wave_stats[wave][r][1] = sum; }
    }
    __syncthreads();
    for (int e = tid; e < nr * kGroup; e += kAttendThreads) {
      const int r = e / kGroup, d = e % kGroup;
      const float M = fmaxf(fmaxf(lds.wave_stats[0][r][0], lds.wave_stats[1][r][0]), fmaxf(lds.wave_stats[2][r][0], lds.wave_stats[3][r][0]));
      const float shift = M == -INFINITY ? 0.f : M;    // every score of the piece is -inf: it weighs nothing in the merge
      const float own = expf(lds.wave_stats[lane & 3][r][0] - shift);        // r is the same in a wave: a factor per lane of a quad
      const float f[4] = {dpp<0x00>(own), dpp<0x55>(own), dpp<0xaa>(own), dpp<0xff>(own)};
      float sum = 0.f, den = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        sum = __fmaf_rn(f[w], lds.sums[w][r][d], sum);
        den = __fmaf_rn(f[w], lds.wave_stats[w][r][1], den);
      }
      const int64_t row = (int64_t)piece * a.q_heads + qh0 + r;
      if (active) a.part[row * kGroup + d] = sum;
      if (active && d == 0) { a.stats[row * 2] = M; a.stats[row * 2 + 1] = den; }
    }
    if (r0 + kMaxRep < rep) stage_queries(r0 + kMaxRep);               // (read ahead of the last barrier)
  }
}

}  // namespace aquakv

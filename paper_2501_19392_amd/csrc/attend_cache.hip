// Attention of one new token per sequence over a cache (Alg. "Inference", Sect. 3.3 of the AQUA-KV paper): over sinks, recovered
// compressed past and recent-token buffer of every sequence of a batch, whatever their lengths, in one launch per layer and one
// more that merges the pieces of several layers.  (Separate launches per sequence, and per kind of token, were 2.5 ms a token for
// 4 sequences of 1020 - 1800 tokens and 8 layers; now 0.55 ms, of which the recovery of the compressed tokens is 0.45 ms.)
//
// The tokens of a sequence are numbered through, [sinks | compressed | recent], and cut into pieces of 64; a workgroup takes
// one piece of one kv head for all its query heads, so the split follows the tokens there are and no sequence waits for another.
// A token's place in memory is picked row by row, and its number is its position for the rotary embedding.
// All sums run in a fixed order, so a call gives the same bits every time.
#include "attend_piece.h"

namespace aquakv {
namespace {

constexpr int kThreads = kAttendThreads;

template <typename T>
__global__ __launch_bounds__(kThreads, 4) void attend_cache_kernel(const AttendCacheArgs) {
  __shared__ AttendLds lds;
  attend_piece<T>(*(AttendCacheParam*)(const void*)__builtin_amdgcn_kernarg_segment_ptr(), (int)blockIdx.x, (int)threadIdx.x, true, lds);
}

// out[layer][b, qh, d] = sum_c e^(m_c - M) part_c / sum_c e^(m_c - M) l_c over the pieces c of sequence b, M = max_c m_c.
// blockIdx = (b * q_heads + qh, layer); thread (k = tid / 32, l = tid % 32) takes dims 4 l ... of pieces k, k + 8, ...
// Bound by the latency of what it reads: the first kHeld pieces of a thread (2048 tokens of a sequence) are requested at once, before
// the maximum over them is known, four more at a time after that.  8 layers of 32 query heads, 4 sequences of 1800 tokens 4.9 us,
// 6 layers of 24 query heads, 8000 tokens 7.7 us; with a value per thread, every other piece each, 6.8 and 11.8 us.
constexpr int kClasses = kThreads / 32, kHeld = 4;
__global__ __launch_bounds__(kThreads) void merge_pieces_kernel(const MergeArgs a) {
  __shared__ __align__(16) float red[kClasses][kGroup];
  __shared__ float top[kClasses], den[kClasses];
  const int b = blockIdx.x / a.q_heads, qh = blockIdx.x % a.q_heads;
  const int k = threadIdx.x >> 5, l = threadIdx.x & 31;
  const int c0 = a.pieces.first[b] + k, c1 = a.pieces.first[b + 1];
  const float* const part = a.part + blockIdx.y * a.part_layer + qh * kGroup + 4 * l;
  const float* const stats = a.stats + blockIdx.y * a.stats_layer + qh * 2;
  f32x4 x[kHeld];
  f32x2 st[kHeld];                                     // maximum, sum of the weights
  const auto request = [&](int c) {
#pragma unroll
    for (int u = 0; u < kHeld; ++u) {
      st[u] = f32x2{-INFINITY, 0.f};
      x[u] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (c + u * kClasses < c1) {
        const int64_t row = (int64_t)(c + u * kClasses) * a.q_heads;
        st[u] = *reinterpret_cast<const f32x2*>(stats + row * 2);
        x[u] = *reinterpret_cast<const f32x4*>(part + row * kGroup);
      }
    }
  };
  request(c0);
  float m = -INFINITY;
#pragma unroll
  for (int u = 0; u < kHeld; ++u) m = fmaxf(m, st[u].x);
#pragma unroll 4
  for (int c = c0 + kHeld * kClasses; c < c1; c += kClasses) m = fmaxf(m, stats[(int64_t)c * a.q_heads * 2]);
  if (l == 0) top[k] = m;
  __syncthreads();
  float M = top[0];
#pragma unroll
  for (int w = 1; w < kClasses; ++w) M = fmaxf(M, top[w]);
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
  float weight = 0.f;
  for (int c = c0;;) {
#pragma unroll
    for (int u = 0; u < kHeld; ++u) {
      if (c + u * kClasses >= c1) break;
      const float e = expf(st[u].x - M);
#pragma unroll
      for (int i = 0; i < 4; ++i) sum[i] = __fmaf_rn(e, x[u][i], sum[i]);
      weight = __fmaf_rn(e, st[u].y, weight);
    }
    c += kHeld * kClasses;
    if (c >= c1) break;
    request(c);
  }
  *reinterpret_cast<f32x4*>(&red[k][4 * l]) = sum;
  if (l == 0) den[k] = weight;
  __syncthreads();
  const int d = threadIdx.x;
  if (d < kGroup) {
    float total = red[0][d], by = den[0];
#pragma unroll
    for (int w = 1; w < kClasses; ++w) { total += red[w][d]; by += den[w]; }
    a.out[blockIdx.y][((a.seq0 + b) * a.q_heads + qh) * kGroup + d] = total / by;
  }
}

}  // namespace

hipError_t launch_attend_cache(int dtype, const AttendCacheArgs& a, hipStream_t stream) {
  const unsigned blocks = attend_workgroups(a, kThreads);
  if (blocks == 0) return hipSuccess;
  if (dtype == kBF16) attend_cache_kernel<bf16_t><<<blocks, kThreads, 0, stream>>>(a);
  else attend_cache_kernel<float><<<blocks, kThreads, 0, stream>>>(a);
  return hipGetLastError();
}

hipError_t launch_merge_pieces(const MergeArgs& a, int layers, hipStream_t stream) {
  if (layers == 0 || a.pieces.n_seq == 0) return hipSuccess;
  merge_pieces_kernel<<<dim3((unsigned)(a.pieces.n_seq * a.q_heads), (unsigned)layers), kThreads, 0, stream>>>(a);
  return hipGetLastError();
}

}  // namespace aquakv

// Least-squares fit of a linear predictor (Alg. "Calibration" of the AQUA-KV paper, Sect. 3.2):
//   W = argmin || [x0 | x1] W^T - Y ||^2 + lambda ||W||^2,   lambda = rate * trace(X^T X) / d_in,
// through the normal equations in fp64:  G = X^T X + lambda I,  R = Y^T X,  G = L L^T (Cholesky),
// Z = R L^-T, W = Z L^-1 rounded to the storage dtype.  With an intercept, X and Y are centred first (the Gram
// products of the centred data are those of the raw data minus T mean mean^T) and b = mean(Y) - W mean(X).
//
// Everything is tiled in 64 x 64 blocks of doubles and multiplied on the fp64 matrix cores.  The Gram products stream the
// tokens once per output tile; work is dealt out in equal shares of (tile, 32 tokens) pieces, so that the last round of
// tiles does not leave CUs idle.  The right-hand sides are rows below G: the blocked factorisation carries them along (the
// forward substitution costs no launches of its own), and the backward substitution leaves W in the layout it is stored in.
// Both take one launch per block column: a launch brings everything behind the column that was finished last up to date, and
// the workgroups of the next column go on to finish that one.
// The Gram products of bf16 data are formed in integers where sizes and data allow (exact_gram.hip), those of fp32 data and all others here.
// 65536 tokens, 2048 inputs, 1024 outputs: 8.3 ms for the Gram products, 0.75 ms forward (23 us a launch), 0.30 ms backward;
// 13.6 ms and 10.9 ms for the rest with scalar 64 x 64 factorisations and five launches per block column.
#include "device_utils.h"
#include "kernels.h"

#include <type_traits>
#include <utility>

namespace aquakv {
namespace {

constexpr int kNb = 64;                      // block size of every tile
constexpr int kFitThreads = 256;

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

// v_mfma_f64_16x16x4_f64: D[16 x 16] += A[16 x 4] B[4 x 16]; lane l holds A[l % 16][l / 16] and B[l / 16][l % 16], i.e. one
// double each, and D[4 v + l / 16][l % 16] in register v.
__device__ __forceinline__ f64x4 mfma64(double a, double b, f64x4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

// ------------------------------------------------------------------ Gram products
// Tiles 0 .. nd (nd + 1) / 2 - 1 are the lower triangle of G(i, j) = sum_t X[t, 64 i ...] X[t, 64 j ...], j <= i, row by
// row; the nr * nd tiles behind are R(i, j) = sum_t Y[t, 64 i ...] X[t, 64 j ...].  X is the concatenation [x0 | x1]; d0
// is a multiple of 64, so a tile's 64 columns come from one of the two.
//
// The steps of all tiles, tile after tile, are cut into gridDim.x equal ranges, one per CU, that all end together, where one
// workgroup per tile leaves most CUs idle in the last round.  A range is at least a tile long (gram_grid), so a tile is shared
// by at most two workgroups: they add their sums to the zeroed output, and 0 + a + b is the same number in either order.
//
// Each of the 8 waves (two per SIMD) multiplies whole 64 x 64 tiles, over an eighth of the tokens: of a step's 8 kGramRows<T>
// tokens wave w takes kGramRows<T>, which it loads itself, as they are stored, straight into its own ring of LDS, four steps
// ahead; so the waves never wait for one another, and an operand that was read and converted to doubles serves four
// instructions.  With the tokens as the contracted index both operands are read from the token-major rows as they lie: lane l
// takes the four columns 4 (l % 16) ... of token l / 16 at once, one for each row (column) block, a step ahead of their use.
// The eight sums are added through LDS at the end of a tile, in a fixed order.
// Bound by the fp64 matrix cores (64 cycles per instruction), which the conversions share: v_cvt_f64_f32 runs in the same
// units.  65536 tokens, 2048 inputs, 1024 outputs (558 GFLOP): 8.3 ms (67 TFLOP/s, 90% of the cycles in the matrix cores);
// 13.6 ms with a workgroup of 4 waves per tile (1040 tiles on 768 places), quarters of the tile per wave and a single stage of
// doubles in LDS.
constexpr int kGramWaves = 8, kGramStages = 4;
constexpr int kGramPieceBytes = 2048;                                        // a wave's rows of one operand: 2 x 64 lanes x 16 bytes
constexpr int kGramStageBytes = 2 * kGramPieceBytes;
constexpr int kGramRingBytes = kGramStages * kGramStageBytes;                // per wave
template <typename T> constexpr int kGramRows = kGramPieceBytes / (kNb * (int)sizeof(T));       // 16 bf16, 8 fp32
constexpr int gram_grid(int tiles) { return tiles >= 256 ? 256 : tiles; }

template <typename T> struct Quad;                                           // four neighbouring elements of a row
template <> struct Quad<bf16_t> {
  u32x2 u;
  __device__ __forceinline__ void get(double (&v)[4]) const {
    v[0] = (double)__uint_as_float(u.x << 16);
    v[1] = (double)__uint_as_float(u.x & 0xffff0000u);
    v[2] = (double)__uint_as_float(u.y << 16);
    v[3] = (double)__uint_as_float(u.y & 0xffff0000u);
  }
};
template <> struct Quad<float> {
  f32x4 u;
  __device__ __forceinline__ void get(double (&v)[4]) const { v[0] = (double)u.x; v[1] = (double)u.y; v[2] = (double)u.z; v[3] = (double)u.w; }
};

template <typename T>
__global__ __launch_bounds__(kGramWaves * 64) void gram_kernel(const T* __restrict__ x0, int d0, const T* __restrict__ x1, int d1,
                                                               const T* __restrict__ Y, int d_out, int64_t tokens,
                                                               double* __restrict__ G, double* __restrict__ R, const int* __restrict__ wanted) {
  if (wanted != nullptr && *wanted == 0) return;
  typedef __attribute__((address_space(3))) unsigned char* lptr_t;
  typedef const __attribute__((address_space(1))) char* gptr_t;
  constexpr int kRows = kGramRows<T>, kRowBytes = kNb * (int)sizeof(T);      // 128 or 256 bytes
  constexpr int kSums = kNb * kNb / 64;                                      // sums per lane of a wave
  __shared__ __attribute__((aligned(16))) unsigned char smem[kGramWaves * kGramRingBytes];
  static_assert(sizeof(smem) == kGramWaves / 2 * kSums * 64 * sizeof(double), "the exchange: half of the waves' sums");
  const int d = d0 + d1, nd = d / kNb, nr = d_out / kNb;
  const int n_sym = nd * (nd + 1) / 2;
  constexpr int kStepRows = kGramWaves * kRows;
  const int64_t steps = (tokens + kStepRows - 1) / kStepRows;
  const int64_t total = steps * (n_sym + nr * nd);
  const auto cut = [&](int64_t b) { return total / gridDim.x * b + total % gridDim.x * b / gridDim.x; };
  int64_t at = cut(blockIdx.x);
  const int64_t end = cut(blockIdx.x + 1);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int fr = lane & 15, fk = lane >> 4;
  constexpr int kLaneRows = 1024 / kRowBytes;                                // token rows per load instruction
  const int lrow = lane / (kRowBytes / 16), lcol = lane % (kRowBytes / 16) * 16;
  unsigned char* const ring = smem + wave * kGramRingBytes;
  const lptr_t ring3 = (lptr_t)ring;
  const auto uniform_ptr = [](const char* p) {
    const uint64_t u = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u), hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
    return (gptr_t)(((uint64_t)hi << 32) | lo);
  };
  double* const exchange = reinterpret_cast<double*>(smem);                  // [wave % 4][sum][lane]
  while (at < end) {
    int tile = (int)(at / steps);
    const int64_t first = at % steps;
    const int64_t last = first + (end - at) < steps ? first + (end - at) : steps;      // steps [first, last) of the tile
    at += last - first;
    const bool is_r = tile >= n_sym;
    int ti = 0, tj;
    if (is_r) {
      tile -= n_sym;
      ti = tile / nd; tj = tile % nd;
    } else {
      while (tile > ti) { tile -= ti + 1; ++ti; }                            // row ti of the triangle holds ti + 1 tiles
      tj = tile;
    }
    const auto column = [&](int block, const char*& p, int& ld) {            // 64 columns of X
      const int col = block * kNb;
      p = reinterpret_cast<const char*>(col < d0 ? x0 + col : x1 + (col - d0));
      ld = (col < d0 ? d0 : d1) * (int)sizeof(T);
    };
    const char *pa, *pb;
    int lda, ldb;
    column(tj, pb, ldb);
    if (is_r) { pa = reinterpret_cast<const char*>(Y + ti * kNb); lda = d_out * (int)sizeof(T); }
    else column(ti, pa, lda);
    // step s into its stage; steps behind the range load its last one again, which keeps the count of loads in flight, and rows
    // behind the tokens the last token
    const auto load = [&](int64_t s, int stage) {
      int64_t t0 = (s < last ? s : last - 1) * kStepRows + wave * kRows;
      t0 = t0 < tokens ? t0 : tokens - 1;
      const int rows = (int)(tokens - 1 - t0 < kRows ? tokens - 1 - t0 : kRows);
      const gptr_t base_a = uniform_ptr(pa + t0 * lda), base_b = uniform_ptr(pb + t0 * ldb);
#pragma unroll
      for (int n = 0; n < kRows / kLaneRows; ++n) {
        const int row = lrow + n * kLaneRows < rows ? lrow + n * kLaneRows : rows;
        const lptr_t dst = ring3 + (stage * kGramStageBytes + n * 1024);
        __builtin_amdgcn_global_load_lds(base_a + (uint32_t)(__umul24(row, lda) + lcol), dst, 16, 0, 0);
        __builtin_amdgcn_global_load_lds(base_b + (uint32_t)(__umul24(row, ldb) + lcol), dst + kGramPieceBytes, 16, 0, 0);
      }
    };
    constexpr int kLoads = 2 * (kRows / kLaneRows);
    f64x4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
    struct Frags { Quad<T> a[kRows / 4], b[kRows / 4]; };
    const auto read = [&](int stage, Frags& f) {
      const unsigned char* const p = ring + stage * kGramStageBytes + fk * kRowBytes + fr * 4 * (int)sizeof(T);
#pragma unroll
      for (int k = 0; k < kRows / 4; ++k) {
        f.a[k] = *reinterpret_cast<const Quad<T>*>(p + 4 * k * kRowBytes);
        f.b[k] = *reinterpret_cast<const Quad<T>*>(p + 4 * k * kRowBytes + kGramPieceBytes);
      }
    };
    // the MFMAs of four tokens, among them the conversions of the next four; CHECKED: tokens from `valid` on are none
    const auto multiply = [&](const Frags& f, auto checked, int64_t valid) {
      double a[2][4], b[2][4];
      const auto convert = [&](int k) {
        f.a[k].get(a[k & 1]);
        f.b[k].get(b[k & 1]);
        if (decltype(checked)::value && 4 * k + fk >= valid) {
#pragma unroll
          for (int e = 0; e < 4; ++e) a[k & 1][e] = b[k & 1][e] = 0.0;
        }
      };
      convert(0);
#pragma unroll
      for (int k = 0; k < kRows / 4; ++k) {
#pragma unroll
        for (int m = 0; m < 16; ++m) {
          acc[m >> 2][m & 3] = mfma64(a[k & 1][m >> 2], b[k & 1][m & 3], acc[m >> 2][m & 3]);
          if (m == 3 && k + 1 < kRows / 4) convert(k + 1);
        }
      }
    };
    // Step s, whose rows are in `now`: its stage is free for step s + kGramStages; step s + 1 has landed and is read.
    int stage = 0;
    const auto step = [&](int64_t s, const Frags& now, Frags& next, auto checked) {
      __builtin_amdgcn_s_waitcnt(0x0070 | (kLoads * (kGramStages - 2) & 15) | (kLoads * (kGramStages - 2) >> 4 << 14));
      asm volatile("" ::: "memory");
      const int following = stage == kGramStages - 1 ? 0 : stage + 1;
      read(following, next);
      load(s + kGramStages, stage);
      multiply(now, checked, tokens - s * kStepRows - wave * kRows);
      stage = following;
    };
    Frags f[2];
#pragma unroll
    for (int n = 0; n < kGramStages; ++n) load(first + n, n);
    __builtin_amdgcn_s_waitcnt(0x0070 | (kLoads * (kGramStages - 1) & 15) | (kLoads * (kGramStages - 1) >> 4 << 14));
    asm volatile("" ::: "memory");
    read(0, f[0]);
    const int64_t whole = last * kStepRows <= tokens ? last : last - 1;      // a step that ends behind the tokens is the tile's last
    int64_t s = first;
    for (; s + 1 < whole; s += 2) {
      step(s, f[0], f[1], std::false_type{});
      step(s + 1, f[1], f[0], std::false_type{});
    }
    for (; s < last; ++s) {                                                  // at most two
      step(s, f[0], f[1], std::true_type{});
      f[0] = f[1];
    }
    // the eight sums: waves 4 - 7 give theirs to waves 0 - 3, whose four then are added by all
    __builtin_amdgcn_s_waitcnt(0x0070);                                      // nothing is on its way into the rings any more
    __syncthreads();
    double* const mine = exchange + (wave & 3) * (kSums * 64) + lane;
    if (wave >= 4) {
#pragma unroll
      for (int e = 0; e < kSums; ++e) mine[e * 64] = acc[e >> 4][e & 3][(e >> 2) & 3];
    }
    __syncthreads();
    if (wave < 4) {
#pragma unroll
      for (int e = 0; e < kSums; ++e) mine[e * 64] += acc[e >> 4][e & 3][(e >> 2) & 3];
    }
    __syncthreads();
    // sum e = 16 i + 4 v + j of lane l is the output at row 16 v + 4 (l / 16) + i, column 4 (l % 16) + j of the tile
    double* const out = (is_r ? R : G) + (int64_t)(ti * kNb + 4 * fk) * d + tj * kNb + 4 * fr;          // both have d columns
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const int i = wave >> 1, v = (wave & 1) * 2 + n;
      double sum[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const double* const p = exchange + (16 * i + 4 * v + j) * 64 + lane;
        sum[j] = ((p[0] + p[kSums * 64]) + p[2 * kSums * 64]) + p[3 * kSums * 64];
      }
      double* const o = out + (int64_t)(16 * v + i) * d;
      if (last - first == steps) {
        reinterpret_cast<f64x2*>(o)[0] = f64x2{sum[0], sum[1]};
        reinterpret_cast<f64x2*>(o)[1] = f64x2{sum[2], sum[3]};
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) unsafeAtomicAdd(o + j, sum[j]);
      }
    }
    __syncthreads();                                                         // the exchange has been read: the rings are free
  }
}

__global__ __launch_bounds__(256) void zero_kernel(f64x2* __restrict__ p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = f64x2{0.0, 0.0};
}

// ------------------------------------------------------------------ intercept (centred regression)
// Column means of [X | Y]: blockIdx.x = 64-column block (the first d_in / 64 blocks are X, the rest Y); 4 strands of
// tokens per column, added in a fixed order.
template <typename T>
__global__ __launch_bounds__(kFitThreads) void column_mean_kernel(const T* __restrict__ x0, int d0, const T* __restrict__ x1,
                                                                  int d1, const T* __restrict__ Y, int d_out, int64_t tokens,
                                                                  double* __restrict__ mean) {
  __shared__ double part[4][kNb];
  const int d_in = d0 + d1;
  const int c0 = blockIdx.x * kNb;
  const T* p;
  int ld;
  if (c0 < d0) { p = x0 + c0; ld = d0; }
  else if (c0 < d_in) { p = x1 + (c0 - d0); ld = d1; }
  else { p = Y + (c0 - d_in); ld = d_out; }
  const int c = threadIdx.x & 63, strand = threadIdx.x >> 6;
  double s = 0.0;
  for (int64_t t = strand; t < tokens; t += 4) s += (double)static_cast<float>(p[t * ld + c]);
  part[strand][c] = s;
  __syncthreads();
  if (strand == 0) mean[c0 + c] = (((part[0][c] + part[1][c]) + part[2][c]) + part[3][c]) / (double)tokens;
}

// G -= T mx mx^T, R -= T my mx^T: the Gram products of the centred data from those of the raw data
__global__ void centre_kernel(double* __restrict__ G, double* __restrict__ R, const double* __restrict__ mean, int d_in,
                              int d_out, double tokens) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t ng = (int64_t)d_in * d_in;
  if (e < ng) {
    const int i = (int)(e / d_in), j = (int)(e % d_in);
    G[e] -= tokens * mean[i] * mean[j];
  } else if (e < ng + (int64_t)d_in * d_out) {
    const int64_t f = e - ng;
    const int o = (int)(f / d_in), i = (int)(f % d_in);
    R[f] -= tokens * mean[d_in + o] * mean[i];
  }
}

// b[o] = my[o] - sum_i W[o][i] mx[i], fp32 out; one workgroup per output; NaN after a failed factorisation
__global__ __launch_bounds__(kFitThreads) void intercept_kernel(const double* __restrict__ S, const double* __restrict__ mean,
                                                                int d_in, float* __restrict__ bias, const int* __restrict__ status) {
  __shared__ double part[kFitThreads];
  const int o = blockIdx.x;
  double s = 0.0;
  for (int i = threadIdx.x; i < d_in; i += kFitThreads) s += S[(int64_t)o * d_in + i] * mean[i];
  part[threadIdx.x] = s;
  __syncthreads();
  for (int w = kFitThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) bias[o] = *status != 0 ? __uint_as_float(0x7fc00000u) : (float)(mean[d_in + o] - part[0]);
}

// G[i][i] += rate * trace(G) / d (one block; the trace is summed in a fixed order); clears the status word
__global__ __launch_bounds__(kFitThreads) void ridge_kernel(double* __restrict__ G, int d, double rate, int* status) {
  __shared__ double part[kFitThreads];
  if (threadIdx.x == 0) *status = 0;
  double s = 0.0;
  for (int i = threadIdx.x; i < d; i += kFitThreads) s += G[(int64_t)i * d + i];
  part[threadIdx.x] = s;
  __syncthreads();
  for (int w = kFitThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  const double lam = rate * part[0] / d;
  for (int i = threadIdx.x; i < d; i += kFitThreads) G[(int64_t)i * d + i] += lam;
}

// ------------------------------------------------------------------ factorisation and substitution
// Row stride 66 doubles: a fragment read (16 rows x 2 consecutive columns per 32 lanes) covers all 64 banks once.
constexpr int kBlkLd = kNb + 2;
typedef double Block[kNb][kBlkLd];
__device__ __forceinline__ void load_block(Block& dst, const double* __restrict__ src, int64_t ld) {
#pragma unroll
  for (int n = 0; n < kNb * kNb / 2 / kFitThreads; ++n) {
    const int e = n * kFitThreads + threadIdx.x, r = e >> 5, c = (e & 31) * 2;
    *reinterpret_cast<f64x2*>(&dst[r][c]) = *reinterpret_cast<const f64x2*>(src + r * ld + c);
  }
}

// Wave w's 16 x 64 strip of a block (rows 16 w ...) as four 16 x 16 accumulators: element (4 v + l / 16, l % 16) of
// sub-block b in b[b][v] of lane l.
struct Strip { f64x4 b[4]; };
__device__ __forceinline__ void load_strip(Strip& s, const double* p, int64_t ld) {      // p: the block's first element
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int v = 0; v < 4; ++v) s.b[b][v] = p[(16 * wave + 4 * v + (lane >> 4)) * ld + 16 * b + (lane & 15)];
}
__device__ __forceinline__ void store_strip(double* p, int64_t ld, const Strip& s) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int v = 0; v < 4; ++v) p[(16 * wave + 4 * v + (lane >> 4)) * ld + 16 * b + (lane & 15)] = s.b[b][v];
}
__device__ __forceinline__ void put_sub_block(Block& dst, const f64x4& x, int b) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int v = 0; v < 4; ++v) dst[16 * wave + 4 * v + (lane >> 4)][16 * b + (lane & 15)] = x[v];
}
// this wave's LDS writes are visible to its other lanes (a strip is touched by one wave only)
__device__ __forceinline__ void wave_sync_lds() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

// s -= A B^T (TRANS) or A B, with A's rows of this wave
template <bool TRANS>
__device__ __forceinline__ void subtract_product(Strip& s, const Block& A, const Block& B) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int fr = lane & 15, fk = lane >> 4;
#pragma unroll
  for (int k = 0; k < kNb; k += 4) {
    const double a = -A[16 * wave + fr][k + fk];
#pragma unroll
    for (int b = 0; b < 4; ++b) s.b[b] = mfma64(a, TRANS ? B[16 * b + fr][k + fk] : B[k + fk][16 * b + fr], s.b[b]);
  }
}

// A factored diagonal block keeps L_kk's 16 x 16 sub-blocks below the diagonal ones and, above them, the inverses of the four on
// the diagonal, which is the form the substitutions need those in.
__device__ __forceinline__ constexpr int inv_row(int b) { return 16 * (b >> 1); }
__device__ __forceinline__ constexpr int inv_col(int b) { return 32 + 16 * (b & 1); }

// X <- X L^-T on the strip, sub-block after sub-block: X_b = (X_b - sum_{m < b} X_m L(b, m)^T) Linv_b^T.  `x`: this wave's rows
// of a block of LDS to turn the results into operands of the next products.
__device__ __forceinline__ void solve_forward(Strip& s, Block& x, const Block& l) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int fr = lane & 15, fk = lane >> 4;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    f64x4 acc = s.b[b];
#pragma unroll
    for (int k = 0; k < 16 * b; k += 4) acc = mfma64(-x[16 * wave + fr][k + fk], l[16 * b + fr][k + fk], acc);
    put_sub_block(x, acc, b);
    wave_sync_lds();
    f64x4 out = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 16; k += 4)
      out = mfma64(x[16 * wave + fr][16 * b + k + fk], l[inv_row(b) + fr][inv_col(b) + k + fk], out);
    wave_sync_lds();
    put_sub_block(x, out, b);
    wave_sync_lds();
    s.b[b] = out;
  }
}
// X <- X L^-1 on the strip, last sub-block first: X_b = (X_b - sum_{m > b} X_m L(m, b)) Linv_b
__device__ __forceinline__ void solve_backward(Strip& s, Block& x, const Block& l) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int fr = lane & 15, fk = lane >> 4;
#pragma unroll
  for (int b = 3; b >= 0; --b) {
    f64x4 acc = s.b[b];
#pragma unroll
    for (int k = 16 * (b + 1); k < kNb; k += 4) acc = mfma64(-x[16 * wave + fr][k + fk], l[k + fk][16 * b + fr], acc);
    put_sub_block(x, acc, b);
    wave_sync_lds();
    f64x4 out = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 16; k += 4)
      out = mfma64(x[16 * wave + fr][16 * b + k + fk], l[inv_row(b) + k + fk][inv_col(b) + fr], out);
    wave_sync_lds();
    put_sub_block(x, out, b);
    wave_sync_lds();
    s.b[b] = out;
  }
}

// 1 / p and 1 / sqrt(p) of a normal p > 0 to the last place or two: the hardware's estimate (better than 2^-20) and two Newton
// steps.  The library's division and square root take several times as many dependent instructions, and the pivots of a block
// wait for one another.
__device__ __forceinline__ double reciprocal(double p) {
  double y = __builtin_amdgcn_rcp(p);
  y = __fma_rn(__fma_rn(-p, y, 1.0), y, y);
  return __fma_rn(__fma_rn(-p, y, 1.0), y, y);
}
__device__ __forceinline__ double reciprocal_root(double p) {
  double y = __builtin_amdgcn_rsq(p);
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    const double e = __fma_rn(-(p * y), y, 1.0);                // 1 - p y^2
    y = __fma_rn(y * e, __fma_rn(e, 0.375, 0.5), y);
  }
  return y;
}

// element N of the lane's group of 16
template <int N> __device__ __forceinline__ double broadcast(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x150 + N, 0xf, 0xf, true);           // row_newbcast
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), 0x150 + N, 0xf, 0xf, true);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Factorisation of one 16 x 16 sub-block by one wave without a trip to LDS: lane l holds row l % 16 in v (every group of 16
// lanes the same) and, in w, columns 4 (l / 16) ... of that row of the identity, which the row operations take to the inverse of
// the factor.  The columns are eliminated with their pivots as they stand, A(i, j) -= A(i, c) A(j, c) / p_c; the roots, which
// nothing waits for, come at the end: row i of the inverse gets its 1 / sqrt(p_i).
struct SubBlock {
  double v[16], w[4], p;
  bool ok;
  template <int C, int... J> __device__ __forceinline__ void column(int r, std::integer_sequence<int, J...>) {
    const double pivot = broadcast<C>(v[C]);
    ok = ok && pivot > 0.0;
    if (r == C) p = pivot;
    const double f = v[C] * reciprocal(pivot);
    const double g = r > C ? f : 0.0;
    ((J > C ? (void)(v[J] = __fma_rn(-f, broadcast<J>(v[C]), v[J])) : (void)0), ...);
#pragma unroll
    for (int q = 0; q < 4; ++q) w[q] = __fma_rn(-g, broadcast<C>(w[q]), w[q]);
  }
  template <int... C> __device__ __forceinline__ void columns(int r, std::integer_sequence<int, C...> all) {
    (column<C>(r, all), ...);
  }
};

// Cholesky factorisation of the block in `a` (lower triangle given) by the whole workgroup, 16 columns at a time: the diagonal
// sub-block by every wave for itself, the sub-blocks below and the trailing ones on the matrix cores, a block row per wave.
// Returns false, in every thread, if a pivot is not positive.
__device__ __forceinline__ bool factor_block(Block& a) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int fr = lane & 15, fk = lane >> 4;
  for (int b = 0; b < 4; ++b) {
    SubBlock s;
#pragma unroll
    for (int m = 0; m < 16; ++m) s.v[m] = a[16 * b + fr][16 * b + m];
#pragma unroll
    for (int q = 0; q < 4; ++q) s.w[q] = fr == 4 * fk + q ? 1.0 : 0.0;
    s.p = 1.0;
    s.ok = true;
    s.columns(fr, std::make_integer_sequence<int, 16>{});
    if (!s.ok) return false;                                   // the same in every lane of every wave
    const double root = reciprocal_root(s.p);
    if (wave == 0) {
#pragma unroll
      for (int q = 0; q < 4; ++q) a[inv_row(b) + fr][inv_col(b) + 4 * fk + q] = s.w[q] * root;
    }
    __syncthreads();
    if (wave > b) {                                            // sub-block (wave, b) below the diagonal one
      f64x4 out = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int k = 0; k < 16; k += 4)
        out = mfma64(a[16 * wave + fr][16 * b + k + fk], a[inv_row(b) + fr][inv_col(b) + k + fk], out);
      wave_sync_lds();
      put_sub_block(a, out, b);
    }
    __syncthreads();
    if (wave > b) {                                            // sub-blocks (wave, n), b < n <= wave
      for (int n = b + 1; n <= wave; ++n) {
        f64x4 acc;
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = a[16 * wave + 4 * q + fk][16 * n + fr];
#pragma unroll
        for (int k = 0; k < 16; k += 4) acc = mfma64(-a[16 * wave + fr][16 * b + k + fk], a[16 * n + fr][16 * b + k + fk], acc);
        put_sub_block(a, acc, n);
      }
    }
    __syncthreads();
  }
  return true;
}

// M: nb block rows of G, then nr of R, all of nb block columns.  Block column k < j is final (k = j - 1 >= 0); this launch
//   finishes column j:      M(i, j) <- (M(i, j) - M(i, k) M(j, k)^T) L_jj^-T, i > j   (the first nb + nr - j workgroups)
//   and updates the others: M(i, n) <- M(i, n) - M(i, k) M(n, k)^T, j < n < nb, i >= n.
// Every workgroup of column j factors the diagonal block for itself, which costs no time (they would wait for it otherwise);
// the one of i = j stores the factor.  Not in place, since the others read the diagonal block meanwhile: L_jj goes to block
// (j, j + 1), above the diagonal.  The factor of the last column is needed by its own workgroups only, which go on to the
// first step of the backward substitution, R(r, nb - 1) <- R(r, nb - 1) L^-1.
// Bound by latency: load, product of two blocks, 64 pivots in turn (about 9 us), substitution.
__global__ __launch_bounds__(kFitThreads, 2) void forward_kernel(double* __restrict__ M, int d, int nb, int nr, int j, int* status) {
  __shared__ Block A, B;
  const int k = j - 1;
  const int panel = nb + nr - j;
  const auto at = [&](int bi, int bj) { return M + (int64_t)bi * kNb * d + bj * kNb; };
  int i, n;
  if ((int)blockIdx.x < panel) {
    i = j + blockIdx.x; n = j;
  } else {
    int p = blockIdx.x - panel;
    const int m = nb - 1 - j;                                  // columns to update; R's rows come first
    if (p < m * nr) { i = nb + p / m; n = j + 1 + p % m; }
    else {
      p -= m * nr;
      int row = 0;
      while (p > row) { p -= row + 1; ++row; }
      i = j + 1 + row; n = j + 1 + p;
    }
  }
  Strip x, diag;
  load_strip(x, at(i, n), d);
  if (n == j) load_strip(diag, at(j, j), d);
  if (k >= 0) {
    load_block(A, at(i, k), d);
    load_block(B, at(n, k), d);
    __syncthreads();
    subtract_product<true>(x, A, B);
    if (n == j) subtract_product<true>(diag, B, B);
    __syncthreads();
  }
  if (n == j) {
#pragma unroll
    for (int b = 0; b < 4; ++b) put_sub_block(B, diag.b[b], b);
    __syncthreads();
    if (!factor_block(B)) {
      if (threadIdx.x == 0) *status = j + 1;                   // every workgroup of the column finds it
      return;
    }
    if (i == j) {
      if (j + 1 < nb) {
        load_strip(x, &B[0][0], kBlkLd);
        store_strip(at(j, j + 1), d, x);
      }
      return;
    }
    solve_forward(x, A, B);
    if (j == nb - 1) solve_backward(x, A, B);
  }
  store_strip(at(i, n), d, x);
}

// Column k + 1 of R is final; this launch updates the columns before it, R(r, i) <- R(r, i) - R(r, k + 1) L(k + 1, i), i <= k,
// and finishes column k: R(r, k) <- R(r, k) L_kk^-1.  blockIdx.x = (k - i) nr + r.
__global__ __launch_bounds__(kFitThreads, 2) void backward_kernel(const double* __restrict__ G, double* __restrict__ R, int d, int nr,
                                                               int k) {
  __shared__ Block A, B;
  const int i = k - (int)blockIdx.x / nr, r = blockIdx.x % nr;
  Strip x;
  load_strip(x, R + (int64_t)r * kNb * d + i * kNb, d);
  load_block(A, R + (int64_t)r * kNb * d + (k + 1) * kNb, d);
  load_block(B, G + (int64_t)(k + 1) * kNb * d + i * kNb, d);
  __syncthreads();
  subtract_product<false>(x, A, B);
  if (i == k) {
    __syncthreads();
    load_block(B, G + (int64_t)k * kNb * d + (k + 1) * kNb, d);
    __syncthreads();
    solve_backward(x, A, B);
  }
  store_strip(R + (int64_t)r * kNb * d + i * kNb, d, x);
}

// fp64 -> storage dtype with one rounding (nearest even).  bf16: the double is first taken to fp32 towards zero with
// the discarded bits ORed into the last place (round to odd), which the final rounding to 8 bits cannot see.
template <typename T> __device__ __forceinline__ T round_from_double(double v);
template <> __device__ __forceinline__ float round_from_double<float>(double v) { return (float)v; }
template <> __device__ __forceinline__ bf16_t round_from_double<bf16_t>(double v) {
  float f = __double2float_rz(v);
  if ((double)f != v && f == f) f = __uint_as_float(__float_as_uint(f) | 1u);
  return static_cast<bf16_t>(f);
}

// W = S rounded to the storage dtype; W64 (nullable) receives the unrounded solution.  A failed factorisation (status != 0)
// yields NaNs.
template <typename T>
__global__ void round_kernel(const double* __restrict__ S, int64_t n, T* __restrict__ W, double* __restrict__ W64,
                             const int* __restrict__ status) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const double v = *status != 0 ? __longlong_as_double(0x7ff8000000000000ll) : S[e];
  W[e] = round_from_double<T>(v);
  if (W64 != nullptr) W64[e] = v;
}

template <typename T>
hipError_t fit(int64_t tokens, const T* x0, int d0, const T* x1, int d1, const T* Y, int d_out, double rate, T* W, double* W64,
               float* bias, void* workspace, hipStream_t stream) {
  const int d = d0 + d1;
  const int nb = d / kNb, nr = d_out / kNb;
  double* G = static_cast<double*>(workspace);
  double* R = G + (size_t)d * d;                               // block rows nb ... of the same matrix
  double* mean = R + (size_t)d * d_out;
  int* status = reinterpret_cast<int*>(mean + d + d_out);
  const int tiles = nb * (nb + 1) / 2 + nb * nr;
  const int64_t n_all = (int64_t)d * (d + d_out);
  // bf16: in integers, and by gram_kernel only if the data turns out not to allow it (the flag behind the status word)
  const bool exact = std::is_same<T, bf16_t>::value && exact_gram_fits(tokens, d0, d1, d_out);
  int* const flag = status + 1;
  zero_kernel<<<1024, 256, 0, stream>>>(reinterpret_cast<f64x2*>(G), (n_all + d + d_out) / 2 + 1);      // the whole workspace
  if (exact)
    if (const hipError_t e = launch_exact_gram(tokens, x0, d0, x1, d1, Y, d_out, G, mean, flag, stream)) return e;
  gram_kernel<T><<<gram_grid(tiles), kGramWaves * 64, 0, stream>>>(x0, d0, x1, d1, Y, d_out, tokens, G, R, exact ? flag : nullptr);
  if (bias != nullptr) {       // intercept: regress the centred Y on the centred X
    column_mean_kernel<T><<<nb + nr, kFitThreads, 0, stream>>>(x0, d0, x1, d1, Y, d_out, tokens, mean);
    centre_kernel<<<(unsigned)((n_all + 255) / 256), 256, 0, stream>>>(G, R, mean, d, d_out, (double)tokens);
  }
  ridge_kernel<<<1, kFitThreads, 0, stream>>>(G, d, rate, status);
  for (int j = 0; j < nb; ++j) {
    const int m = nb - 1 - j;
    const int updated = j > 0 ? m * (m + 1) / 2 + m * nr : 0;
    forward_kernel<<<nb + nr - j + updated, kFitThreads, 0, stream>>>(G, d, nb, nr, j, status);
  }
  for (int k = nb - 2; k >= 0; --k) backward_kernel<<<(k + 1) * nr, kFitThreads, 0, stream>>>(G, R, d, nr, k);
  if (bias != nullptr) intercept_kernel<<<d_out, kFitThreads, 0, stream>>>(R, mean, d, bias, status);
  const int64_t n = (int64_t)d * d_out;
  round_kernel<T><<<(unsigned)((n + 255) / 256), 256, 0, stream>>>(R, n, W, W64, status);
  return hipGetLastError();
}

}  // namespace

size_t fit_workspace_bytes(int d_in, int d_out) {
  // G, R / solution, column means of [X | Y], status word
  return ((size_t)d_in * d_in + (size_t)d_in * d_out + d_in + d_out) * sizeof(double) + 16;
}

hipError_t launch_fit_predictor(int dtype, int64_t tokens, const void* x0, int d0, const void* x1, int d1, const void* Y,
                                int d_out, double rate, void* W, double* W64, float* bias, void* workspace,
                                hipStream_t stream) {
  if (dtype == kBF16)
    return fit(tokens, static_cast<const bf16_t*>(x0), d0, static_cast<const bf16_t*>(x1), d1, static_cast<const bf16_t*>(Y),
               d_out, rate, static_cast<bf16_t*>(W), W64, bias, workspace, stream);
  return fit(tokens, static_cast<const float*>(x0), d0, static_cast<const float*>(x1), d1, static_cast<const float*>(Y), d_out,
             rate, static_cast<float*>(W), W64, bias, workspace, stream);
}

}  // namespace aquakv

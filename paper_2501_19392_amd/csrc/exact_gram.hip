// The Gram products of the least-squares fit (calibrate.hip) over bf16 data, exactly, on the 8-bit integer matrix cores.
//
// bf16 values have 8 significant bits, and those of one column mostly lie within a few powers of two of the largest one.  With the
// column's unit set 13 binades below its largest exponent almost every value is an integer q of at most 22 bits, which three signed
// digits of 8 bits hold: q = d0 + 2^8 d1 + 2^16 d2.  The nine digit products of two columns are summed in int32 by
// v_mfma_i32_32x32x32_i8 and put together in int64, where no sum of up to 2^20 tokens rounds or overflows, and which comes out the same in any
// order of additions.  (Products of floating-point matrices by way of slices whose products are exact: Ozaki, Ogita, Oishi and Rump, Numerical
// Algorithms 59, 2012; on integer matrix units: Ootomo, Ozaki and Yokota, 2024.)  Values more than 13 binades below their column's largest (of Gaussian columns 3 to 6 in 10000) are rounded to the
// nearest q; what is left of them is listed per column and enters in fp64 with the single rounding of the sum (finish_kernel).  So the result is closer
// to the exact one than a sum in fp64, whose every step rounds.  Where a list would overflow, the lists cost more than the integers gain
// (list_cost_limit), or a column holds infinities, NaNs or nothing but values too small to be scaled, a flag sends the whole product to the fp64
// kernel of calibrate.hip.
//
// A fit of 65536 tokens, 2048 inputs and 1024 outputs 9.23 -> 3.24 ms (Gram products 8.1 -> 2.2: the products 1.89, the two passes that find
// scales and lists 0.17, finish_kernel 0.14), 65536 x 1024 inputs 3.56 -> 1.35, 16384 x 2048 3.13 -> 1.62, 4096 x 1024 0.71 -> 0.61.
#include "device_utils.h"
#include "kernels.h"

#include <type_traits>
#include <utility>

namespace aquakv {
namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

constexpr int kBinades = 13;                 // between the unit of a column and its largest exponent: |q| <= 255 << 13
constexpr int kGramXcds = 8;

// [x0 | x1 | Y] as one row of d + d_out columns; 128 neighbouring ones, from a multiple of 128, lie in one of the three
struct Columns {
  const bf16_t *x0, *x1, *Y;
  int d0, d1, d_out;
  __device__ __forceinline__ const bf16_t* at(int c, int& ld) const {
    if (c < d0) { ld = d0; return x0 + c; }
    c -= d0;
    if (c < d1) { ld = d1; return x1 + c; }
    ld = d_out;
    return Y + (c - d1);
  }
};

// The lists of a fit: entries of 4 bytes in the blocks of G above the diagonal ones, which hold nothing until the factorisation.  A row of
// a 64 x 64 block is a piece of 128 entries; column c of n has pieces c, c + n, c + 2 n ...
constexpr int kPieceEntries = 128, kMaxListed = 1024;
__host__ __device__ __forceinline__ int listed_room(int d, int columns) {
  const int nb = d / 64, pieces = nb * (nb - 1) / 2 * 64 / columns;
  return pieces * kPieceEntries < kMaxListed ? pieces * kPieceEntries : kMaxListed;
}
__device__ __forceinline__ uint32_t* listed(double* G, int d, int columns, int c, int n) {
  const int piece = c + n / kPieceEntries * columns, block = piece >> 6;
  int bj = (int)((1.f + sqrtf(8.f * (float)block + 1.f)) * 0.5f);      // block column bj holds blocks bj (bj - 1) / 2 ...
  while (bj * (bj - 1) / 2 > block) --bj;
  while (bj * (bj + 1) / 2 <= block) ++bj;
  const int bi = block - bj * (bj - 1) / 2;
  return reinterpret_cast<uint32_t*>(G + (int64_t)(bi * 64 + (piece & 63)) * d + bj * 64) + n % kPieceEntries;
}

// A column's largest magnitude (the bits of the value without its sign) gives the exponent of its scale
__device__ __forceinline__ int top_exponent(uint32_t largest) { return (int)(largest >> 7) > 1 ? (int)(largest >> 7) : 1; }
__device__ __forceinline__ int scale_exponent(uint32_t largest) {      // q = value * 2^this
  const int e = 134 + kBinades - top_exponent(largest);
  return e < 127 ? e : 127;                                            // (only for columns of zeros: see list_kernel)
}
__device__ __forceinline__ float scale_of(uint32_t largest) { return __uint_as_float((uint32_t)(127 + scale_exponent(largest)) << 23); }
// value * scale rounded to an integer, plus 2^23 + kDigits in the low bits of the float: bytes d0 + 128, d1 + 128, d2 + 64
constexpr float kMagic = 8388608.f + 4227200.f;                        // 4227200 = 0x408080
__device__ __forceinline__ float rounded(float value, float scale) { return __builtin_fmaf(value, scale, kMagic); }

constexpr int kScanRows = 16;
// one workgroup: 128 columns, 8 a lane, of kScanRows tokens in each of 16 strands
template <typename F>
__device__ __forceinline__ void scan(const Columns& x, int64_t tokens, F&& f) {
  const int lane = threadIdx.x & 15, strand = threadIdx.x >> 4;        // 16 lanes x 8 columns, 16 strands of tokens
  const int c = (int)blockIdx.x * 128 + lane * 8;
  int ld;
  const bf16_t* p = x.at((int)blockIdx.x * 128, ld) + lane * 8;
  const int64_t t0 = (int64_t)blockIdx.y * (16 * kScanRows) + strand;
  f(c, p, ld, t0);
}

// largest[c] = the largest magnitude of column c (zero before)
__global__ __launch_bounds__(256) void largest_kernel(const Columns x, int64_t tokens, uint32_t* __restrict__ largest) {
  __shared__ uint32_t most[16][128 + 4];
  uint32_t m[8] = {};
  scan(x, tokens, [&](int, const bf16_t* p, int ld, int64_t t0) {
#pragma unroll
    for (int n = 0; n < kScanRows; ++n) {
      const int64_t t = t0 + n * 16 < tokens ? t0 + n * 16 : tokens - 1;
      const u32x4 v = *reinterpret_cast<const u32x4*>(p + t * ld);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t lo = v[k] & 0x7fffu, hi = (v[k] >> 16) & 0x7fffu;
        m[2 * k] = lo > m[2 * k] ? lo : m[2 * k];
        m[2 * k + 1] = hi > m[2 * k + 1] ? hi : m[2 * k + 1];
      }
    }
  });
  const int lane = threadIdx.x & 15, strand = threadIdx.x >> 4;
#pragma unroll
  for (int k = 0; k < 8; ++k) most[strand][lane * 8 + k] = m[k];
  __syncthreads();
  if (threadIdx.x < 128) {
    uint32_t all = 0;
    for (int s = 0; s < 16; ++s) all = most[s][threadIdx.x] > all ? most[s][threadIdx.x] : all;
    atomicMax(&largest[blockIdx.x * 128 + threadIdx.x], all);
  }
}

// The values that their q does not hold exactly, or may not: tokens to the column's list, in any order.  flag: the fp64 kernel's work.
//
// A workgroup counts its 256 tokens' entries of each column in LDS and takes their places in the list with one atomic per column, so that
// data whose lists overflow (a column that holds an infinity lists all its finite values) cost no more than others.  With an atomic per
// entry, 65536 tokens, 2048 inputs, 1024 outputs, ms, fp64 sums alone / before / now: half of the columns small but for one token 9.21 / 28.9 /
// 9.36, a tenth of all values small 9.21 / 12.8 / 9.39, an infinity in one column 8.90 / 9.99 / 9.07; nothing but lists of 50 entries 3.38 / 3.43,
// 4096 tokens, 256 inputs, 128 outputs 0.255 / 0.204.
__global__ __launch_bounds__(256, 8) void list_kernel(const Columns x, int64_t tokens, const uint32_t* __restrict__ largest,
                                                   uint32_t* __restrict__ count, double* __restrict__ G, int* __restrict__ flag) {
  __shared__ int entries[128], first[128];                             // of the workgroup's columns; where they start in the lists, or -1
  if (threadIdx.x < 128) entries[threadIdx.x] = 0;
  __syncthreads();
  const int d = x.d0 + x.d1, columns = d + x.d_out, room = listed_room(d, columns);
  scan(x, tokens, [&](int c, const bf16_t* p, int ld, int64_t t0) {
    uint32_t least[8];                                                 // magnitudes below, but zero, are listed
    bool bad = false;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint32_t m = largest[c + k];
      const int e = top_exponent(m);
      bad |= e == 255 || (m != 0 && 134 + kBinades - e > 127);
      least[k] = (uint32_t)(e > kBinades ? e - kBinades : 0) << 7;
    }
    if (bad) *flag = 1;
    uint32_t listed_rows[8] = {};                                      // bit n: row n
#pragma unroll 1
    for (int n0 = 0; n0 < kScanRows; n0 += 8) {                        // (16 rows in flight take 88 registers, five waves per SIMD and not eight)
#pragma unroll
      for (int n = n0; n < n0 + 8; ++n) {
        const int64_t t = t0 + n * 16;
        const u32x4 v = *reinterpret_cast<const u32x4*>(p + (t < tokens ? t : tokens - 1) * ld);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const uint32_t m = (k & 1 ? v[k >> 1] >> 16 : v[k >> 1]) & 0x7fffu;
          listed_rows[k] |= (m < least[k] && m != 0 && t < tokens ? 1u : 0u) << n;
        }
      }
    }
    const int column = (int)(threadIdx.x & 15) * 8;
    int at[8] = {};                                                    // place among the workgroup's entries of the column
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (listed_rows[k] != 0) at[k] = atomicAdd(&entries[column + k], __popc(listed_rows[k]));
    __syncthreads();
    if (threadIdx.x < 128) {
      const int own = (int)blockIdx.x * 128 + (int)threadIdx.x, n = entries[threadIdx.x];
      const int from = n != 0 ? (int)atomicAdd(&count[own], (uint32_t)n) : 0;
      first[threadIdx.x] = from + n <= room ? from : -1;
      if (from + n > room) *flag = 1;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int from = first[column + k];
      if (from < 0) continue;
      for (uint32_t rows = listed_rows[k]; rows != 0; rows &= rows - 1)
        *listed(G, d, columns, c + k, from + at[k]++) = (uint32_t)(t0 + (__ffs((int)rows) - 1) * 16);
    }
  });
}

// Lists in the order of their tokens, so that the sums over them do not depend on the order of arrival: one workgroup per column.  The
// first workgroup finds what finish_kernel will take for all of them; the product is the fp64 kernel's work if that is more than `most`.
struct ListCost {
  unsigned long long walks;                                            // entries, each once for every block that goes through its list
  uint32_t four;                                                       // entries of four neighbouring columns (a wave's in a block)
};
__global__ __launch_bounds__(256) void sort_kernel(int d, int columns, const uint32_t* __restrict__ count, double* __restrict__ G,
                                                   int* __restrict__ flag, const ListCost most) {
  __shared__ uint32_t token[kMaxListed];
  if (blockIdx.x == 0) {
    __shared__ ListCost all;
    if (threadIdx.x == 0) all = {0, 0};
    __syncthreads();
    const uint32_t nd = d / 64, nr = (columns - d) / 64;
    ListCost own = {0, 0};
#pragma unroll 4
    for (int c = 4 * threadIdx.x; c < columns; c += 4 * 256) {
      const u32x4 v = *reinterpret_cast<const u32x4*>(count + c);
      const uint32_t n = v.x + v.y + v.z + v.w;
      own.walks += (unsigned long long)n * (c < d ? nd + 1 + nr : nd);
      own.four = n > own.four ? n : own.four;
    }
    atomicAdd(&all.walks, own.walks);
    atomicMax(&all.four, own.four);
    __syncthreads();
    if (threadIdx.x == 0 && (all.walks > most.walks || all.four > most.four)) *flag = 1;
    return;
  }
  const int c = (int)blockIdx.x - 1, n = (int)count[c];
  if (n < 2 || n > listed_room(d, columns)) return;                    // (more than the room: the flag is set, and nothing reads the list)
  for (int i = threadIdx.x; i < n; i += 256) token[i] = *listed(G, d, columns, c, i);
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += 256) {
    int rank = 0;
    for (int k = 0; k < n; ++k) rank += token[k] < token[i];
    *listed(G, d, columns, c, rank) = token[i];
  }
}

// ------------------------------------------------------------------ the products
// 128 x 128 outputs per tile: the lower triangle of X^T X by blocks, then Y^T X, in bands of four block rows, column after column, so that
// neighbouring tiles share their rows and columns.  Every XCD has an equal share of neighbouring tiles: its 32 workgroups take whole ones as
// long as there are 32 and go through the tokens side by side, reading each column block once from beyond their L2; the tiles
// left over are cut into 32 equal ranges of steps.  Sums are added to the zeroed output with integer atomics.
//
// Step: 64 tokens of the tile's 256 columns.  Wave w takes 16 tokens of 128 columns (two neighbouring ones per lane) from memory, a step
// ahead, turns them into digits (2.6 instructions a value: one fma that scales and rounds, the bytes of four tokens transposed) and stores them
// to LDS as the operands that the instructions read: 32 columns x 32 tokens of a digit are 1 KiB, lane l column l % 32, tokens 16 (l / 32) ...;
// of 32 columns the even ones come first, which makes 16 lanes' stores contiguous.  Each of the 8 waves (two per SIMD) multiplies 64 x 32
// outputs: five accumulators (powers of 2^8) of two blocks, 160 registers, 36 instructions of 32 cycles.  Nothing else would fit beside a second
// set of operands, so a register is read again as soon as its last instruction has been issued, and all other work is placed between the
// matrix instructions, with the step's one barrier six of them behind the last store (8 % fewer cycles than next to it).
// 16384 tokens, 2048 inputs, 1024 outputs: matrix cores busy in 0.65 of the cycles, at 1.90 GHz, 2.58 POPS; 65536 tokens 2.70 POPS.  A form with operands
// read at the start of their 32 tokens: busy in 0.52, at 2.0 GHz.
// int32 holds 65535 tokens of any digits: segments of at most kMaxSteps steps.
constexpr int kMfma = 0x008, kValu = 0x002, kLdsRead = 0x100, kLdsWrite = 0x200;      // kinds for sched_group_barrier
constexpr int kExactThreads = 512, kStepTokens = 64, kMaxSteps = 512, kTile = 128;
constexpr int kUnit = 1024, kStageBytes = 2 * 4 * 3 * 2 * kUnit;       // operand, 32-column block, digit, 32 tokens

// what comes behind the matrix instructions of a step (36), which are two or three for an operand that is read again
template <int N> __device__ __forceinline__ void behind_mfma() {
  __builtin_amdgcn_sched_group_barrier(kMfma, 1, 0);
  if constexpr (N == 5 || N == 11 || N == 29) __builtin_amdgcn_sched_group_barrier(kLdsRead, 2, 0);
  if constexpr (N == 13 || N == 15 || N == 31 || N == 33) __builtin_amdgcn_sched_group_barrier(kLdsRead, 1, 0);
  if constexpr (N == 17 || N == 35) __builtin_amdgcn_sched_group_barrier(kLdsRead, 3, 0);
  if constexpr (N >= 12 && N < 18) __builtin_amdgcn_sched_group_barrier(kLdsWrite, 1, 0);
  __builtin_amdgcn_sched_group_barrier(kValu, N < 13 ? 7 : 5, 0);
}
template <int FIRST, int... N> __device__ __forceinline__ void instruction_order(std::integer_sequence<int, N...>) { (behind_mfma<FIRST + N>(), ...); }

__global__ __launch_bounds__(kExactThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void exact_gram_kernel(
    const Columns x, int64_t tokens, const uint32_t* __restrict__ largest, double* __restrict__ G, const int* __restrict__ flag) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[2 * kStageBytes];
  if (*flag != 0) return;
  const int d = x.d0 + x.d1;
  const int nx = d / kTile, ny = x.d_out / kTile;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int steps = (int)((tokens + kStepTokens - 1) / kStepTokens);
  const uint32_t lane4 = 4 * lane;
  const int wm = wave >> 2, wn = wave & 3;                             // multiplied: 64 rows, 32 columns
  const int operand = wave >> 2, quarter = wave & 3;                   // converted: rows or columns of the tile, 16 tokens of a step
  // where this lane's even column goes: unit (operand, lane / 16, digit, quarter / 2)
  unsigned char* const put = smem + ((operand * 4 + (lane >> 4)) * 6 + (quarter >> 1)) * kUnit + (quarter & 1) * 512 + (lane & 15) * 16;
  const unsigned char* const get_a = smem + wm * 2 * 6 * kUnit + lane * 16;
  const unsigned char* const get_b = smem + (4 + wn) * 6 * kUnit + lane * 16;

  const auto run = [&](int tile, int first, int last) {
    int bi = 0, bj = 0;
    {                                                                  // bands of four block rows, those of G first
      const int n_sym = nx * (nx + 1) / 2;
      int rest = tile < n_sym ? tile : tile - n_sym;
      const int rows = tile < n_sym ? nx : ny, sym = tile < n_sym;
      int band = 0;
      for (;; band += 4) {
        const int h = rows - band < 4 ? rows - band : 4;
        const int n = sym ? h * band + h * (h + 1) / 2 : h * nx;
        if (rest < n) break;
        rest -= n;
      }
      const int h = rows - band < 4 ? rows - band : 4;
      if (!sym || rest < h * band) {
        bj = rest / h;
        bi = band + rest % h;
      } else {
        rest -= h * band;
        int col = 0;
        while (rest >= h - col) { rest -= h - col; ++col; }
        bj = band + col;
        bi = band + col + rest;
      }
      if (!sym) bi += nx;
    }
    int ld;
    const int c0 = (operand == 0 ? bi : bj) * kTile;
    const bf16_t* const base = x.at(c0, ld);
    const uint32_t row_bytes = (uint32_t)ld * sizeof(bf16_t);
    const float scale0 = scale_of(largest[c0 + 2 * lane]), scale1 = scale_of(largest[c0 + 2 * lane + 1]);
    // the range's tokens as a buffer (512 steps of rows of 16 KiB: its bytes fit 30 bits); reads behind it return zeros
    const int64_t token = (int64_t)first * kStepTokens, behind = (int64_t)last * kStepTokens < tokens ? (int64_t)last * kStepTokens : tokens;
    const __amdgpu_buffer_rsrc_t rows =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(base + token * ld), 0, (int)((uint32_t)(behind - token) * row_bytes), 0x00020000);
    uint32_t raw[16];
    const auto load = [&](int s, int from, int n) {                    // rows from ... of a step's 16
      uint32_t row = ((uint32_t)(s - first) * kStepTokens + quarter * 16 + from) * row_bytes;
#pragma unroll
      for (int r = 0; r < n; ++r) {
        raw[from + r] = __builtin_amdgcn_raw_buffer_load_b32(rows, (int)(row + lane4), 0, 0);
        row += row_bytes;
      }
    };
    // digits of tokens 4 g ... : one word of each digit for both columns
    const auto convert = [&](int g, u32x4 (&out)[2][3]) {
      const uint32_t* const r = raw + 4 * g;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        uint32_t w[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
          w[k] = __float_as_uint(rounded(__uint_as_float(e ? r[k] & 0xffff0000u : r[k] << 16), e ? scale1 : scale0));
        const uint32_t lo01 = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u), lo23 = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u);
        const uint32_t hi = __builtin_amdgcn_perm(w[1], w[0], 0x0c0c0602u) | __builtin_amdgcn_perm(w[3], w[2], 0x06020c0cu);
        out[e][0][g] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u) ^ 0x80808080u;
        out[e][1][g] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u) ^ 0x80808080u;
        out[e][2][g] = (hi + 0x40404040u) ^ 0x80808080u;               // (bytes of 32 to 96: no carry)
      }
    };
    const auto store = [&](int stage, const u32x4 (&out)[2][3]) {
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int p = 0; p < 3; ++p) *reinterpret_cast<u32x4*>(put + stage * kStageBytes + p * 2 * kUnit + e * 256) = out[e][p];
    };
    const auto barrier = [] {                                          // this wave's LDS accesses are done; loads stay in flight
      __builtin_amdgcn_s_waitcnt(0xc07f);
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    };
    i32x16 acc[2][5];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int o = 0; o < 5; ++o)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[m][o][e] = 0;

    i32x4 a[2][3], b[3];                                               // operands of the next 32 tokens' instructions
    const auto read_a = [&](int stage, int kb, int p) {
#pragma unroll
      for (int m = 0; m < 2; ++m) a[m][p] = *reinterpret_cast<const i32x4*>(get_a + stage * kStageBytes + ((m * 3 + p) * 2 + kb) * kUnit);
    };
    const auto read_b = [&](int stage, int kb, int p) {
      b[p] = *reinterpret_cast<const i32x4*>(get_b + stage * kStageBytes + (p * 2 + kb) * kUnit);
    };
    u32x4 out[2][3];
    load(first, 0, 16);
#pragma unroll
    for (int g = 0; g < 4; ++g) convert(g, out);
    store(0, out);
    load(first + 1, 0, 16);
    barrier();
#pragma unroll
    for (int p = 0; p < 3; ++p) { read_b(0, 0, p); read_a(0, 0, p); }
    convert(0, out);
    convert(1, out);
    load(first + 2, 0, 8);
    int stage = 0;
    // the instructions of 32 tokens with digit pa of the rows; operands are read again, for the 32 tokens after these, once they are used
    const auto multiply = [&](int kb, int pa) {
      const int from = kb == 0 ? stage : stage ^ 1;
#pragma unroll
      for (int pb = 0; pb < 3; ++pb) {
#pragma unroll
        for (int m = 0; m < 2; ++m)
          acc[m][pa + pb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[m][pa], b[pb], acc[m][pa + pb], 0, 0, 0);
        if (pa == 2) read_b(from, kb ^ 1, pb);
      }
      read_a(from, kb ^ 1, pa);
    };
    for (int s = first; s < last; ++s) {
      multiply(0, 0);
      convert(2, out);
      load(s + 2, 8, 4);
      multiply(0, 1);
      convert(3, out);
      load(s + 2, 12, 4);
      store(stage ^ 1, out);
      multiply(0, 2);
      convert(0, out);
      load(s + 3, 0, 4);
#pragma unroll
      for (int pb = 0; pb < 3; ++pb)
#pragma unroll
        for (int m = 0; m < 2; ++m) acc[m][pb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[m][0], b[pb], acc[m][pb], 0, 0, 0);
      instruction_order<0>(std::make_integer_sequence<int, 24>{});
      __builtin_amdgcn_sched_barrier(0);
      barrier();                                                       // the next step's operands are there
      read_a(stage ^ 1, 0, 0);
      multiply(1, 1);
      convert(1, out);
      load(s + 3, 4, 4);
      multiply(1, 2);
      instruction_order<24>(std::make_integer_sequence<int, 12>{});
      __builtin_amdgcn_sched_barrier(0);
      stage ^= 1;
    }
    barrier();                                                         // the stages are free

    // sums: register r of lane l is row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32 of a block, in the order the columns were put in
    if (!(bi < nx && bj * 2 + (wn >> 1) > bi * 2 + wm)) {              // (above the diagonal: nothing is kept there, but lists)
      const auto placed = [](int p) { return 2 * (p & 15) + (p >> 4); };
      unsigned long long* const to = reinterpret_cast<unsigned long long*>(G) + (int64_t)(bi * kTile + wm * 64) * d + bj * kTile + wn * 32 + placed(lane & 31);
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          long long v = acc[m][4][r];
#pragma unroll
          for (int o = 3; o >= 0; --o) v = v * 256 + acc[m][o][r];
          const int row = placed(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3));
          __hip_atomic_fetch_add(to + (int64_t)(m * 32 + row) * d, (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
  };
  const int n_all = nx * (nx + 1) / 2 + nx * ny;
  const int xcd = blockIdx.x % kGramXcds, w = blockIdx.x / kGramXcds, per = gridDim.x / kGramXcds;
  const int first = n_all * xcd / kGramXcds, n = n_all * (xcd + 1) / kGramXcds - first, whole = n / per * per;
  const int64_t left = (int64_t)(n - whole) * steps, end = left * (w + 1) / per;
  int64_t at = left * w / per;
  for (int i = w; i < whole || at < end;) {
    int tile = first + i, s = 0, last = steps;
    if (i < whole) {
      i += per;
    } else {
      tile = first + whole + (int)(at / steps);
      s = (int)(at % steps);
      last = end - at < steps - s ? s + (int)(end - at) : steps;
      at += last - s;
    }
    for (; s < last; s += kMaxSteps) run(tile, s, last - s < kMaxSteps ? last : s + kMaxSteps);
  }
}

// Integer sums -> fp64, with what the lists hold: in units of the two columns, value = q + r, the sum over tokens of
// value_i value_j is that of q_i q_j (exact), of r_i value_j over i's list and of q_i r_j over j's list.  One workgroup per 64 x 64 block, as in
// gram_kernel (calibrate.hip).  Both sums go through a list with a wave per entry, its 64 partners in the lanes: 140 us for 20 to 40 entries a
// column, 690 with a lane per list of the second sum, whose loads each touch 64 rows.
constexpr int kFinishRows = 4, kFinishUnroll = 8;
__global__ __launch_bounds__(1024) void finish_kernel(const Columns x, const uint32_t* __restrict__ largest, const uint32_t* __restrict__ count,
                                                      double* G, const int* __restrict__ flag) {
  __shared__ double column_part[64][64 + 1];
  if (*flag != 0) return;
  const int d = x.d0 + x.d1, columns = d + x.d_out, nd = d / 64;
  int tile = blockIdx.x, bi = 0, bj;
  if (tile >= nd * (nd + 1) / 2) {
    tile -= nd * (nd + 1) / 2;
    bi = nd + tile / nd; bj = tile % nd;
  } else {
    while (tile > bi) { tile -= bi + 1; ++bi; }
    bj = tile;
  }
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j = bj * 64 + lane, ej = scale_exponent(largest[j]);
  int ldi, ldj;
  const bf16_t* const pi = x.at(bi * 64 & ~127, ldi) + (bi * 64 & 127);
  const bf16_t* const pj = x.at(bj * 64 & ~127, ldj) + (bj * 64 & 127);
  // sum over the list of column c of r_c times the 64 columns at p: their values, or their q (QUANTIZED)
  const auto over_list = [&](int c, const bf16_t* pc, int ldc, const bf16_t* p, int ld, float scale, auto quantized) {
    const int n = (int)count[c], ec = scale_exponent(largest[c]);
    const float sc = scale_of(largest[c]);
    double sum = 0.0;
    for (int k0 = 0; k0 < n; k0 += 64) {                               // a lane fetches an entry, all lanes go through them
      const bool is = k0 + lane < n;
      const int t = (int)*listed(G, d, columns, c, is ? k0 + lane : n - 1);
      const float v = (float)pc[(int64_t)t * ldc];
      const float r = is ? (float)(ldexp((double)v, ec) - (double)(rounded(v, sc) - kMagic)) : 0.f;       // |r| <= 1/2, 8 significant bits
      const int m = n - k0 < 64 ? n - k0 : 64;
      for (int l0 = 0; l0 < m; l0 += kFinishUnroll) {                  // (entries behind the list are its last one with r = 0)
        float other[kFinishUnroll];
#pragma unroll
        for (int l = 0; l < kFinishUnroll; ++l) other[l] = (float)p[(int64_t)__builtin_amdgcn_readlane(t, l0 + l) * ld + lane];
#pragma unroll
        for (int l = 0; l < kFinishUnroll; ++l) {
          const float rl = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(r), l0 + l));
          const float o = decltype(quantized)::value ? rounded(other[l], scale) - kMagic : other[l];
          sum = __fma_rn((double)rl, (double)o, sum);
        }
      }
    }
    return sum;
  };
  // r_i value_j with a row per wave and a column per lane, q_i r_j the other way round, turned in LDS
  double row_part[kFinishRows];
#pragma unroll
  for (int n = 0; n < kFinishRows; ++n) {
    const int w = wave * kFinishRows + n;
    row_part[n] = ldexp(over_list(bi * 64 + w, pi + w, ldi, pj, ldj, 0.f, std::false_type{}), ej);
    column_part[w][lane] = over_list(bj * 64 + w, pj + w, ldj, pi, ldi, scale_of(largest[bi * 64 + lane]), std::true_type{});
  }
  __syncthreads();
#pragma unroll
  for (int n = 0; n < kFinishRows; ++n) {
    const int w = wave * kFinishRows + n, i = bi * 64 + w;
    double* const o = G + (int64_t)i * d + j;
    const double sum = (double)*reinterpret_cast<const long long*>(o) + (row_part[n] + column_part[lane][w]);
    *o = ldexp(sum, -scale_exponent(largest[i]) - ej);
  }
}

}  // namespace

// Columns in whole tiles of 128, room for lists at all (none below 256 inputs), and as many tokens as int64 sums hold.  Few tokens are not worth
// the launches around the product.  Whole fits, us, fp64 / integers: 2048 inputs and 1024 outputs, 512 tokens 1185 / 1188, 1024 tokens
// 1242 / 1207; 1024 and 1024, 1024 tokens 566 / 574, 1536 tokens 590 / 578; 512 and 512, 2048 tokens 286 / 295, 3072 tokens 319 / 300;
// 256 and 128, 2048 tokens 171 / 160, 3072 tokens 202 / 162.
bool exact_gram_fits(int64_t tokens, int d0, int d1, int d_out) {
  const int64_t columns = (int64_t)d0 + d1 + d_out;
  return (tokens >= 2560 || tokens * columns >= 2600000) && tokens <= (1 << 20) && d0 % kTile == 0 && d1 % kTile == 0 && d_out % kTile == 0 &&
         listed_room(d0 + d1, (int)columns) > 0;
}

// What lists may cost: as much as the integers gain.  The fp64 kernel's and the integer kernel's time differ by 88 ps a token and 64 x 64 block (of
// at least 256 blocks, as many as there are CUs), less 45 us for the launches around the product.  finish_kernel takes 37 ps for an entry of
// a list and block (9.5 ns of a CU), and 0.3 us for an entry of four neighbouring columns, which a wave goes through in turn while its block
// shares the CU with other columns' lists (columns apart from others: 0.1).  Gaussian columns have 2 to 26 entries and stay far below.
// us, n entries in every column, integers / where the line is / behind it, fp64 sums and the passes in vain (without passes): 16384 tokens, 2048
// inputs, 1024 outputs 1625 + 4.3 n / n = 290 / 3250 to 3350 (3130); 4096 tokens, 1024 and 1024 600 + 1.4 n / 51 / 741 to 768 (711); 4096 tokens,
// 256 and 128 162 + 0.9 n / 39 / 252 to 265 (233).  With the room in the lists as the only line 800 entries took 5226 in the first of these.
static ListCost list_cost_limit(int64_t tokens, int d, int d_out) {
  const int64_t nd = d / 64, blocks = nd * (nd + 1) / 2 + nd * (d_out / 64);
  const double us = 88e-6 * (double)tokens * (double)(blocks > 256 ? blocks : 256) - 45.0;
  return us > 0 ? ListCost{(unsigned long long)(us / 37e-6), (uint32_t)(us / 0.3)} : ListCost{0, 0};
}

hipError_t launch_exact_gram(int64_t tokens, const void* x0, int d0, const void* x1, int d1, const void* Y, int d_out, double* G, void* columns,
                             int* flag, hipStream_t stream) {
  const Columns x = {static_cast<const bf16_t*>(x0), static_cast<const bf16_t*>(x1), static_cast<const bf16_t*>(Y), d0, d1, d_out};
  const int d = d0 + d1, all = d + d_out;
  uint32_t* const largest = static_cast<uint32_t*>(columns);
  uint32_t* const count = largest + all;
  const dim3 grid(all / 128, (unsigned)((tokens + 16 * kScanRows - 1) / (16 * kScanRows)));
  largest_kernel<<<grid, 256, 0, stream>>>(x, tokens, largest);
  list_kernel<<<grid, 256, 0, stream>>>(x, tokens, largest, count, G, flag);
  sort_kernel<<<all + 1, 256, 0, stream>>>(d, all, count, G, flag, list_cost_limit(tokens, d, d_out));
  exact_gram_kernel<<<256, kExactThreads, 0, stream>>>(x, tokens, largest, G, flag);
  const int nd = d / 64;
  finish_kernel<<<nd * (nd + 1) / 2 + nd * (d_out / 64), 1024, 0, stream>>>(x, largest, count, G, flag);
  return hipGetLastError();
}

}  // namespace aquakv

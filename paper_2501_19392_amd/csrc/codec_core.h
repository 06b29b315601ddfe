// Building blocks of the backbone quantizer (Sect. 2 "Vector Quantization" of the AQUA-KV
// paper) for one rotation group held by a quad of lanes x 32 values: nearest-grid-point
// search (full, or through the cell table), code packing, and the quantize / dequantize
// bodies shared by the streaming kernels and by the epilogues of the fused predictor kernels.
//
// Nearest grid point.  The definition is a search over all n grid points.  The kernels reach
// the same answer with a 64 x 64 table of square cells over [-4, 4]^2 (border cells are
// unbounded outwards): each cell lists, in ascending order, every grid point that can be
// nearest to some point of the (slightly enlarged) cell -- at most 4 (3 for n = 16), else the
// cell is marked and the lane falls back to the full search.  Only the listed points are
// scored, with the same fp32 expression and the same lowest-index tie rule as the full
// search, so both give identical codes.
//
// Inside the kernels a grid point is named by its "slot" (Slot<NCW>): for n = 16 the byte offset 16 j of its
// entry in the LDS copy of the grid, which still fits a byte of a table entry and is the address the look-up
// needs; for the larger grids the index j itself.
#pragma once
#include <type_traits>

#include "device_utils.h"

namespace aquakv {

constexpr int kCells = 64;                   // table is kCells x kCells
// The cells tile [-R, R]^2 (border cells reach out to infinity).  R = 4 for the grids of 16 and 64 points.  For the
// 256-point grid R = 3.25: where the cell edges fall relative to the grid decides how many cells see more candidates than an
// entry holds, and with R = 4 twelve such cells sit where a Gaussian puts 0.9 % of its mass (so nearly every wave of 1024
// sub-vectors meets one), with R = 3.25 they hold less than 1e-5 of it.
__host__ __device__ constexpr float cell_half_range(int n) { return n == 256 ? 3.25f : 4.0f; }
__host__ __device__ constexpr float cell_scale(int n) { return kCells / (2.0f * cell_half_range(n)); }   // cells per unit
// Table layout (32-bit words): kCells * kCells cell entries, then kOvfLists overflow lists of two words each.
// A cell entry lists up to 4 candidate slots, one per byte from the lowest, ascending, the last one repeated.  A cell
// with more candidates than the kernels score per cell (3 for the 16-point grid, else 4) is CROWDED: its entry is
// crowded_entry(n, L) = 0xFF in the top byte, the largest slot (top = (n - 1) << shift) in the two middle bytes and L
// in the lowest, so that every byte the quantizer may score before it looks at the flag is a slot the grid array can
// be read at (the 16-point grid never scores the top byte, the others hold 256 entries).  L = list << shift names the
// overflow list with the cell's (up to 8) candidates, again one per byte, ascending, last repeated; L = top means no
// list (more than 8 candidates, or no list left): the full search.  An entry is crowded iff it compares >=
// crowded_threshold(n), which no ordinary entry does except, with 256 points, those that list point 255: such cells
// get an overflow list as well, and the ones that list nothing else share list 0.
constexpr int kCellWords = kCells * kCells;
constexpr int kOvfLists = 128;
constexpr int kOvfCand = 8;                  // candidates per overflow list
constexpr int kTableWords = kCellWords + 2 * kOvfLists;
__host__ __device__ constexpr int slot_shift(int n) { return n == 16 ? 4 : 0; }
__host__ __device__ constexpr uint32_t slot_top(int n) { return (uint32_t)(n - 1) << slot_shift(n); }
__host__ __device__ constexpr uint32_t crowded_threshold(int n) {
  return n == 256 ? 0xFF000000u : ((slot_top(n) + 1u) << 24);
}
__host__ __device__ constexpr uint32_t crowded_entry(int n, uint32_t L) {
  return 0xFF000000u | (slot_top(n) << 16) | (slot_top(n) << 8) | L;
}
// lists a grid of n points can name: L = list << shift must stay below top
__host__ __device__ constexpr int ovf_capacity(int n) { return n == 16 ? 15 : (n - 1 < kOvfLists ? n - 1 : kOvfLists); }

// Quantizer ids, the NCW template argument everywhere: 16 / 64 / 256 = a grid of that many points in R^2;
// kRtn2 / kRtn4 = the uniform round-to-nearest backbone with 2 / 4 bits per value (see rtn_quantize_residual).
constexpr int kRtn2 = 2, kRtn4 = 4;
__host__ __device__ constexpr bool is_rtn(int id) { return id < 16; }

// c = code bits per pair of values (a lane holds 16 pairs = 4c code bytes, whatever the quantizer)
template <int NCW> struct CodeBits;
template <> struct CodeBits<kRtn2> { static constexpr int c = 4; };
template <> struct CodeBits<kRtn4> { static constexpr int c = 8; };
template <> struct CodeBits<16> { static constexpr int c = 4; };
template <> struct CodeBits<64> { static constexpr int c = 6; };
template <> struct CodeBits<256> { static constexpr int c = 8; };

// Grid in LDS as (a, b, -(a^2+b^2)/2, unused): argmin ||y - C||^2 = argmax y.C - |C|^2/2.
template <int NCW>
__device__ __forceinline__ void load_codebook(const float* __restrict__ codebook, float4* cb) {
  if constexpr (is_rtn(NCW)) return;          // no grid
  for (int j = threadIdx.x; j < NCW; j += blockDim.x) {
    const float a = codebook[2 * j], b = codebook[2 * j + 1];
    cb[j] = make_float4(a, b, -0.5f * (a * a + b * b), 0.f);
  }
}

__device__ __forceinline__ float score(float y0, float y1, const float4 c) {
  return __fmaf_rn(y0, c.x, __fmaf_rn(y1, c.y, c.z));
}

template <int NCW> struct Slot {
  static constexpr int kShift = slot_shift(NCW);            // slot = j << kShift
};
// the LDS entry of a grid point from its slot (SHIFT = 4: the slot is the byte offset itself)
template <int SHIFT> __device__ __forceinline__ float4 grid_entry(const float4* cb, int slot) {
  return *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(cb) + ((uint32_t)slot << (4 - SHIFT)));
}

// LDS byte offset (inside the table) of the cell of y.  Both coordinates go to [0, 1] over the cells' range, are clamped and
// converted to 16 bits by one instruction, and the top six bits of each are the cell.  Against exact cells the edges sit up
// to 6.1e-5 off (65535 / 65536 and the rounding to nearest), inside the 1e-4 by which the builder enlarges every cell when
// it lists candidates, so the candidate sets still hold and the codes are the same.  Six vector instructions per
// sub-vector; clamping, truncating and combining the coordinates one by one takes nine.
template <int NCW>
__device__ __forceinline__ uint32_t cell_offset(float y0, float y1) {
  const float inv_range = cell_scale(NCW) / kCells;
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  const u16x2 c = __builtin_amdgcn_cvt_pknorm_u16(__fmaf_rn(y0, inv_range, 0.5f), __fmaf_rn(y1, inv_range, 0.5f));
  const uint32_t d = __builtin_bit_cast(uint32_t, c);
  // byte 0: x cell and two spare bits (bits 8 .. 15 of d); byte 1: y cell (bits 26 .. 31 of d)
  return __builtin_amdgcn_perm(d >> 18, d, 0x0c0c0501u) & 0x3ffcu;
}
static_assert(kCells == 64, "six bits per coordinate");
template <int NCW>
__device__ __forceinline__ uint32_t cell_entry(float y0, float y1, const uint32_t* table) {
  return *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(table) + cell_offset<NCW>(y0, y1));
}

// Table search of one sub-vector from the (up to 4, ascending, last one repeated) candidates its cell entry lists, fetched
// beforehand; returns the winner's slot.  If the cell lists too many points (entry >= crowded_threshold) the result is
// void: the caller then redoes the sub-vector from the cell's overflow list, or with the full search (rare; keeps the hot
// path small).
template <int NCW> struct Candidates {
  static constexpr int kCand = NCW == 16 ? 3 : 4;       // the builder marks cells of a 16-point grid with more than 3
  float c[kCand][3];
  __device__ __forceinline__ void fetch(uint32_t e, const float4* cb) {
#pragma unroll
    for (int k = 0; k < kCand; ++k) {
      const float4 g = grid_entry<Slot<NCW>::kShift>(cb, (int)((e >> (8 * k)) & 0xff));
      c[k][0] = g.x; c[k][1] = g.y; c[k][2] = g.z;
    }
  }
  __device__ __forceinline__ int winner(float y0, float y1, uint32_t e) const {
    int slot = e & 0xff;
    float best = score(y0, y1, make_float4(c[0][0], c[0][1], c[0][2], 0.f));
#pragma unroll
    for (int k = 1; k < kCand; ++k) {
      const float s = score(y0, y1, make_float4(c[k][0], c[k][1], c[k][2], 0.f));
      const bool better = s > best;              // duplicates of the last candidate never win
      best = better ? s : best;
      slot = better ? (int)((e >> (8 * k)) & 0xff) : slot;
    }
    return slot;
  }
};

// Full search (the definition: all n points, lowest index wins ties) of N sub-vectors: their slots.
template <int NCW, int N>
__device__ __forceinline__ void search_full(const float (&y)[2 * N], const float4* cb, int (&slot)[N]) {
  float best[N];
  const float4 c0 = cb[0];
#pragma unroll
  for (int k = 0; k < N; ++k) { best[k] = score(y[2 * k], y[2 * k + 1], c0); slot[k] = 0; }
#pragma unroll 1
  for (int j = 1; j < NCW; ++j) {
    const float4 cj = cb[j];
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const float s = score(y[2 * k], y[2 * k + 1], cj);
      const bool better = s > best[k];
      best[k] = better ? s : best[k];
      slot[k] = better ? (j << Slot<NCW>::kShift) : slot[k];
    }
  }
}

// A sub-vector in a crowded cell (low: the entry's lowest byte, naming its overflow list): decided among the list's
// candidates (ascending, strict comparison: the lowest index wins ties, as in the full search), or by the full search
// if the cell has no list.
template <int NCW>
__device__ __forceinline__ int search_crowded(float y0, float y1, uint32_t low, const float4* cb, const uint32_t* table) {
  constexpr int SH = Slot<NCW>::kShift;
  if (low == slot_top(NCW)) {
    const float y[2] = {y0, y1};
    int all[1];
    search_full<NCW, 1>(y, cb, all);
    return all[0];
  }
  const uint32_t* list = table + kCellWords + 2 * (int)(low >> SH);
  int slot = (int)(list[0] & 0xff);
  float best = score(y0, y1, grid_entry<SH>(cb, slot));
  // two rounds of four candidates: the four grid points of a round are fetched together (a loop over single
  // candidates would wait for LDS eight times in a row); rolled, because this path is rare and its size is not
#pragma unroll 1
  for (int rnd = 0; rnd < 2; ++rnd) {
    const uint32_t w = list[rnd];
    float4 c[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) c[k] = grid_entry<SH>(cb, (int)((w >> (8 * k)) & 0xff));
#pragma unroll
    for (int k = 0; k < 4; ++k) {                     // (the first candidate again in round 0: a tie, no change)
      const float sc = score(y0, y1, c[k]);
      const bool better = sc > best;
      best = better ? sc : best;
      slot = better ? (int)((w >> (8 * k)) & 0xff) : slot;
    }
    // a list ends in repeats of its last candidate: no second round if no lane here has more than four
    if (list[1] == (w >> 24) * 0x01010101u) break;
  }
  return slot;
}

// A lane's 16 codes of c bits are 4c contiguous bytes of the group's little-endian bit string, c / 2 words (8 codes: half of
// that).  Adds the code of sub-vector m (compile time) to them, given its slot.
template <int NCW>
__device__ __forceinline__ void pack_code(uint32_t (&d)[4], int m, int slot) {
  constexpr int c = CodeBits<NCW>::c;
  constexpr int SH = Slot<NCW>::kShift;
  if constexpr (c == 4) {
    const int pos = 4 * (m & 7);                     // the index j = slot >> SH goes to bit `pos`
    d[m >> 3] |= pos >= SH ? (uint32_t)slot << (pos - SH) : (uint32_t)slot >> (SH - pos);
  } else {
    static_assert(c == 4 || SH == 0, "slots of the larger grids are indices");
    const int bit = c * m, w = bit >> 5, sh = bit & 31;
    d[w] |= (uint32_t)slot << sh;
    if (sh + c > 32) d[w + 1] |= (uint32_t)slot >> (32 - sh);
  }
}
// N values per lane = c N / 16 code bytes, at position q of the group
template <int NCW, int N>
__device__ __forceinline__ void store_codes(uint8_t* __restrict__ codes, int64_t gid, int q, const uint32_t (&d)[4]) {
  constexpr int c = CodeBits<NCW>::c;
  uint8_t* const at = codes + gid * (kGroup / 2 * c / 8) + q * (N / 16 * c);
  uint32_t* dst = reinterpret_cast<uint32_t*>(at);
  if constexpr (N == 16 && c == 4) {
    dst[0] = d[0];
  } else if constexpr (N == 16 && c == 6) {            // 6 bytes from a multiple of 6: the word among them that is aligned
    const bool odd = q & 1;
    *reinterpret_cast<uint32_t*>(at + (odd ? 2 : 0)) = odd ? (d[0] >> 16) | (d[1] << 16) : d[0];
    *reinterpret_cast<uint16_t*>(at + (odd ? 0 : 4)) = (uint16_t)(odd ? d[0] : d[1]);
  } else if constexpr (N == 16) {
    u32x2 v; v.x = d[0]; v.y = d[1];
    *reinterpret_cast<u32x2*>(dst) = v;
  } else if constexpr (c == 4) {
    u32x2 v; v.x = d[0]; v.y = d[1];
    *reinterpret_cast<u32x2*>(dst) = v;
  } else if constexpr (c == 6) {
    dst[0] = d[0]; dst[1] = d[1]; dst[2] = d[2];
  } else {
    u32x4 v; v.x = d[0]; v.y = d[1]; v.z = d[2]; v.w = d[3];
    *reinterpret_cast<u32x4*>(dst) = v;
  }
}

// the code bytes of a lane, as loaded into (the first dwords of) a register quad -> 16 or 8 indices
template <int NCW, int M>
__device__ __forceinline__ void unpack_codes(const u32x4 raw, int (&idx)[M]) {
  constexpr int c = CodeBits<NCW>::c;
  const uint32_t d[4] = {raw.x, raw.y, raw.z, raw.w};
  if constexpr (c == 4) {
#pragma unroll
    for (int m = 0; m < M; ++m) idx[m] = (d[m >> 3] >> (4 * (m & 7))) & 15;
  } else if constexpr (c == 6) {
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int bit = 6 * m, w = bit >> 5, sh = bit & 31;
      uint32_t x = d[w] >> sh;
      if (sh > 26) x |= d[w + 1] << (32 - sh);
      idx[m] = x & 63;
    }
  } else {
#pragma unroll
    for (int m = 0; m < M; ++m) idx[m] = (d[m >> 2] >> (8 * (m & 3))) & 255;
  }
}

// ... -> the byte offsets of the grid points in the LDS copy of the grid (entries of 16 bytes).  Codes of 4 bits: all of a word moved into the upper
// half of their bytes at once, then one instruction each (a shift and a mask each otherwise; groups across the heads look up 8 heads for every
// value: decode of 2300 tokens 27.8 -> 27.1 us, 32768 227 -> 220; groups of one head within 1 %).
template <int NCW, int M>
__device__ __forceinline__ void unpack_offsets(const u32x4 raw, uint32_t (&off)[M]) {
  if constexpr (CodeBits<NCW>::c == 4) {
    const uint32_t d[2] = {raw.x, raw.y};
#pragma unroll
    for (int w = 0; w < M / 8; ++w) {
      uint32_t even = (d[w] << 4) & 0xf0f0f0f0u, odd = d[w] & 0xf0f0f0f0u;
      asm("" : "+v"(even), "+v"(odd));                       // (the compiler would fold the steps into a shift and a mask each)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        off[8 * w + 2 * k] = (even >> (8 * k)) & 0xffu;
        off[8 * w + 2 * k + 1] = (odd >> (8 * k)) & 0xffu;
      }
    }
  } else {
    int idx[M];
    unpack_codes<NCW>(raw, idx);
#pragma unroll
    for (int m = 0; m < M; ++m) off[m] = (uint32_t)idx[m] << 4;
  }
}
__device__ __forceinline__ float2 grid_point(const float4* cb, uint32_t off) {
  return *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(cb) + off);
}

__device__ __forceinline__ float half_bits_to_float(uint16_t h) {
  return static_cast<float>(__builtin_bit_cast(_Float16, h));
}

// offsets of the lane's grid points -> the points times `scale` (recon_scale(sigma16, lane): the input of the inverse
// transform)
template <int M>
__device__ __forceinline__ void gather_zhat(const uint32_t (&off)[M], float scale, const float4* cb, float (&z)[2 * M]) {
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const float2 cw = grid_point(cb, off[m]);
    z[2 * m] = cw.x * scale;
    z[2 * m + 1] = cw.y * scale;
  }
}

struct Lds {
  float4 cb[256];
  uint32_t table[kTableWords];
};

// The table on its way from memory to LDS through registers (kernels that request it while their LDS is still in
// other use): 16-byte chunk t + i * THREADS for thread t.
template <int THREADS> struct TableRegs {
  static constexpr int kChunks = kTableWords / 4;
  static constexpr int kPerThread = (kChunks + THREADS - 1) / THREADS;
  u32x4 r[kPerThread];
  __device__ __forceinline__ void request(const uint32_t* __restrict__ table) {
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
      const int ch = (int)threadIdx.x + i * THREADS;
      if ((i + 1) * THREADS <= kChunks || ch < kChunks) r[i] = reinterpret_cast<const u32x4*>(table)[ch];
    }
  }
  __device__ __forceinline__ void store(uint32_t* lds_table) const {
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
      const int ch = (int)threadIdx.x + i * THREADS;
      if ((i + 1) * THREADS <= kChunks || ch < kChunks) reinterpret_cast<u32x4*>(lds_table)[ch] = r[i];
    }
  }
};

// ------------------------------------------------------------------ uniform round-to-nearest backbone
// Sect. 4.1 "Backbone quantization" of the paper: b-bit round-to-nearest with per-group normalisation, groups of
// 64 consecutive channels of a token = the 2 x 32 values of a lane pair (quad lanes 0,1 and 2,3).  Per group:
// lo = min(0, min r), hi = max(0, max r), step = (hi - lo) / (2^b - 1) stored as fp16, zero = round(-lo / step),
// code = clamp(round(r / step) + zero, 0, 2^b - 1) with the stored step, rounding half to even.  Stored per
// group: (fp16 step, 16-bit zero point), i.e. `scales` holds two uint16 per group, [T, H, 2 groups, 2].
// Codes: b bits per value in channel order, little-endian: the lane's N values are N b / 8 contiguous bytes.
template <int BITS, int N>
__device__ __forceinline__ void rtn_store_codes(uint8_t* __restrict__ codes, int64_t gid, int q, const uint32_t (&code)[N]) {
  uint32_t* dst = reinterpret_cast<uint32_t*>(codes + gid * (kGroup * BITS / 8) + q * (N / 8 * BITS));
  constexpr int kPerWord = 32 / BITS, kWords = N / kPerWord;
  uint32_t d[kWords] = {};
#pragma unroll
  for (int r = 0; r < N; ++r) d[r / kPerWord] |= code[r] << (BITS * (r % kPerWord));
  if constexpr (kWords == 1) {
    dst[0] = d[0];
  } else if constexpr (kWords == 2) {
    u32x2 v; v.x = d[0]; v.y = d[1];
    *reinterpret_cast<u32x2*>(dst) = v;
  } else {
    u32x4 v; v.x = d[0]; v.y = d[1]; v.z = d[2]; v.w = d[3];
    *reinterpret_cast<u32x4*>(dst) = v;
  }
}

// the lane's code bytes (first dwords of `raw`) and its group's (step, zero) word -> p + (code - zero) * step
template <int BITS, int N>
__device__ __forceinline__ void rtn_reconstruct(const u32x4 raw, uint32_t meta, const float (&p)[N], float (&v)[N]) {
  const uint32_t d[4] = {raw.x, raw.y, raw.z, raw.w};
  constexpr int kPerWord = 32 / BITS;
  const float s16 = half_bits_to_float((uint16_t)(meta & 0xffffu));
  const int zero = (int)(meta >> 16);
#pragma unroll
  for (int r = 0; r < N; ++r) {
    const int code = (int)((d[r / kPerWord] >> (BITS * (r % kPerWord))) & ((1u << BITS) - 1u));
    v[r] = __fmaf_rn((float)(code - zero), s16, p[r]);     // the product is exact: small integer x fp16
  }
}

// the (step, zero) word of the lane's group: two groups of 64 per head, or (WIDE, 8 heads) one group per token
template <bool WIDE = false, int N = 32>
__device__ __forceinline__ uint32_t rtn_load_meta(const uint16_t* __restrict__ scales, int64_t gid, int q) {
  return reinterpret_cast<const uint32_t*>(scales)[WIDE ? gid >> 3 : gid * 2 + q / (64 / N)];
}

// Q of the residuals of the N values this lane holds of head group gid; same contract as quantize_residual below
// (`l`: group_pos, or with WIDE token_pos: the group is then the whole token of 8 heads, one (step, zero) per token).
template <int BITS, bool WIDE = false, int N>
__device__ __forceinline__ void rtn_quantize_residual(float (&v)[N], int l, bool active, int64_t gid,
                                                      uint8_t* __restrict__ codes, uint16_t* __restrict__ scales,
                                                      bool want_hat) {
  const int q = WIDE ? l & (kGroup / N - 1) : l;
  constexpr float kTop = (float)((1 << BITS) - 1);
  float lo = 0.f, hi = 0.f;
#pragma unroll
  for (int r = 0; r < N; ++r) {
    lo = fminf(lo, v[r]);
    hi = fmaxf(hi, v[r]);
  }
  lo = fminf(lo, quad_xor<1>(lo));
  hi = fmaxf(hi, quad_xor<1>(hi));
  if constexpr (N == 16) { lo = fminf(lo, quad_xor<2>(lo)); hi = fmaxf(hi, quad_xor<2>(hi)); }
  if constexpr (WIDE) {
    const auto fold = [&](float lo2, float hi2) { lo = fminf(lo, lo2); hi = fmaxf(hi, hi2); };
    fold(quad_xor<2>(lo), quad_xor<2>(hi));
    fold(octet_mirror(lo), octet_mirror(hi));
    fold(row_xor8(lo), row_xor8(hi));
    const auto far = [&](auto mask) {
      float a = lo, b = lo, c = hi, d = hi;
      swap_lanes<mask()>(a, b);
      swap_lanes<mask()>(c, d);
      lo = fminf(a, b);
      hi = fmaxf(c, d);
    };
    far(std::integral_constant<int, 16>());
    if constexpr (N == 16) far(std::integral_constant<int, 32>());
  }
  const float step = fminf(__fdiv_rn(hi - lo, kTop), 65504.0f);
  const _Float16 s16h = static_cast<_Float16>(step);      // round to nearest even
  const float s16 = static_cast<float>(s16h);
  const bool ok = s16 > 0.f;
  const float inv = ok ? __fdiv_rn(1.0f, s16) : 0.f;
  const float zf = ok ? __builtin_amdgcn_fmed3f(__builtin_rintf(__fdiv_rn(-lo, s16)), 0.f, kTop) : 0.f;
  uint32_t code[N];
#pragma unroll
  for (int r = 0; r < N; ++r)
    code[r] = (uint32_t)__builtin_amdgcn_fmed3f(__builtin_rintf(v[r] * inv) + zf, 0.f, kTop);
  if (active) {
    rtn_store_codes<BITS>(codes, gid, q, code);
    const uint32_t word = (uint32_t)__builtin_bit_cast(uint16_t, s16h) | ((uint32_t)zf << 16);
    if constexpr (WIDE) {
      if (l == 0) reinterpret_cast<uint32_t*>(scales)[gid >> 3] = word;
    } else {
      if (q % (64 / N) == 0) reinterpret_cast<uint32_t*>(scales)[gid * 2 + q / (64 / N)] = word;
    }
  }
  if (want_hat) {
#pragma unroll
    for (int r = 0; r < N; ++r) v[r] = ((float)code[r] - zf) * s16;     // exact: small integer x fp16
  }
}

// ------------------------------------------------------------------ group bodies
// Q of the residuals v = x - p of the N coordinates this lane holds of head group `gid` (= token * H + head).  On exit
// v holds, if `want_hat`, what finish_hat turns into the (unrounded) reconstruction p + Q^-1(codes).  Codes and the
// scale are stored when `active` (inactive lanes only keep the cross-lane exchanges in step).
// `l` is the lane's position inside its rotation group: group_pos for groups of 128 (WIDE = false, one
// scale per head group), token_pos for groups of 1024 = the whole token (WIDE = true, kv_heads = 8, one
// scale per token at scales[gid / 8]).  The code bytes have the same layout in both cases.
// BATCH: sub-vectors searched together.  searched() is called behind the search, when registers are free again.
struct Nothing { __device__ __forceinline__ void operator()() const {} };
template <int NCW, bool WIDE = false, int BATCH = 4, int N, typename Searched = Nothing>
__device__ __forceinline__ void quantize_residual(float (&v)[N], const float (&sf)[N], int l, const float4* cb,
                                                  const uint32_t* table, bool active, int64_t gid,
                                                  uint8_t* __restrict__ codes, uint16_t* __restrict__ scales, bool want_hat,
                                                  Searched&& searched = Nothing()) {
  if constexpr (is_rtn(NCW)) {
    rtn_quantize_residual<NCW, WIDE>(v, l, active, gid, codes, scales, want_hat);
    searched();
    return;
  }
#pragma unroll
  for (int r = 0; r < N; ++r) v[r] *= sf[r];                                             // s * (x - p), exact product
  const int q = WIDE ? l & (kGroup / N - 1) : l;
  Rot<WIDE>::wht(v, l);                                   // w = +-H u (unnormalised, lane sign pending)

  const float ss = Rot<WIDE>::square_sum(v, l);
  // z = w / sqrt(g)  =>  rms(z) = sqrt(sum w^2) / g
  float sigma = __fsqrt_rn(ss) * Rot<WIDE>::kInvG;
  sigma = fminf(sigma, 65504.0f);
  const _Float16 s16h = static_cast<_Float16>(sigma);     // round to nearest even
  const float s16 = static_cast<float>(s16h);
  const float inv = s16 > 0.f ? Rot<WIDE>::sign(l) * __fdiv_rn(Rot<WIDE>::kNorm, s16) : 0.f;   // also undoes the lane sign

  // BATCH sub-vectors at a time: their candidates are in flight together, the codes are packed and (want_hat) the grid
  // points take the place of the rotated values at once, so no more than BATCH slots are ever held.  (All 16 at a time
  // kept the stand-alone kernels at 256 registers, two waves per SIMD.)
  const float rs = recon_scale<WIDE>(s16, l);
  uint32_t words[4] = {0, 0, 0, 0};
#pragma unroll
  for (int m0 = 0; m0 < N / 2; m0 += BATCH) {
    float y[2 * BATCH];
#pragma unroll
    for (int i = 0; i < 2 * BATCH; ++i) y[i] = v[2 * m0 + i] * inv;
    int slot[BATCH];
    if (table != nullptr) {
      uint32_t e[BATCH], top = 0;
#pragma unroll
      for (int k = 0; k < BATCH; ++k) e[k] = cell_entry<NCW>(y[2 * k], y[2 * k + 1], table);
      if constexpr (BATCH > 4) {                     // registers to spare: all candidates requested before any is scored
        Candidates<NCW> cand[BATCH];
#pragma unroll
        for (int k = 0; k < BATCH; ++k) cand[k].fetch(e[k], cb);
#pragma unroll
        for (int k = 0; k < BATCH; ++k) slot[k] = cand[k].winner(y[2 * k], y[2 * k + 1], e[k]);
      } else {
#pragma unroll
        for (int k = 0; k < BATCH; ++k) {
          Candidates<NCW> cand;
          cand.fetch(e[k], cb);
          slot[k] = cand.winner(y[2 * k], y[2 * k + 1], e[k]);
        }
      }
#pragma unroll
      for (int k = 0; k < BATCH; ++k) top = max(top, e[k]);
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(top >= crowded_threshold(NCW)) != 0, 0)) {
#pragma unroll 1
        for (int k = 0; k < BATCH; ++k) {            // rolled: the path is rare, its size is not
          uint32_t ek = 0;
          float y0 = 0.f, y1 = 0.f;
#pragma unroll
          for (int i = 0; i < BATCH; ++i) {          // (no dynamic register indexing)
            ek = k == i ? e[i] : ek; y0 = k == i ? y[2 * i] : y0; y1 = k == i ? y[2 * i + 1] : y1;
          }
          if (ek < crowded_threshold(NCW)) continue;
          const int j = search_crowded<NCW>(y0, y1, ek & 0xffu, cb, table);
#pragma unroll
          for (int i = 0; i < BATCH; ++i) slot[i] = k == i ? j : slot[i];
        }
      }
    } else {
      search_full<NCW, BATCH>(y, cb, slot);          // the definition: scan all n points
    }
#pragma unroll
    for (int k = 0; k < BATCH; ++k) pack_code<NCW>(words, m0 + k, slot[k]);
    if (want_hat) {
#pragma unroll
      for (int k = 0; k < BATCH; ++k) {
        const float2 cw = *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(cb) + ((uint32_t)slot[k] << (4 - Slot<NCW>::kShift)));
        v[2 * (m0 + k)] = cw.x * rs;
        v[2 * (m0 + k) + 1] = cw.y * rs;
      }
    }
  }
  if (active) {
    store_codes<NCW, N>(codes, gid, q, words);
    if (l == 0) scales[WIDE ? gid >> 3 : gid] = __builtin_bit_cast(uint16_t, s16h);
  }
  searched();
  if (want_hat) Rot<WIDE>::iwht(v, l);
}
// the reconstruction from quantize_residual's v and the prediction
template <int NCW, int N>
__device__ __forceinline__ void finish_hat(float (&v)[N], const float (&sf)[N], const float (&p)[N]) {
#pragma unroll
  for (int r = 0; r < N; ++r) v[r] = is_rtn(NCW) ? v[r] + p[r] : __fmaf_rn(v[r], sf[r], p[r]);
}
// Q(x - p): on entry v = x, on exit p + Q^-1(codes) if `want_hat`
template <int NCW, bool WIDE = false, int BATCH = 4, int N>
__device__ __forceinline__ void quantize_group(float (&v)[N], const float (&p)[N], const float (&sf)[N], int l,
                                               const float4* cb, const uint32_t* table, bool active, int64_t gid,
                                               uint8_t* __restrict__ codes, uint16_t* __restrict__ scales, bool want_hat) {
#pragma unroll
  for (int r = 0; r < N; ++r) v[r] -= p[r];
  quantize_residual<NCW, WIDE, BATCH>(v, sf, l, cb, table, active, gid, codes, scales, want_hat);
  if (want_hat) finish_hat<NCW>(v, sf, p);
}

// the lane's share of a group's codes (and of its scales) as the kernels hold them between request and use
struct CodeWords { u32x4 code; uint32_t scale; };   // scale: fp16 bits (grids) or (step, zero point) (round-to-nearest)

// requests the code bytes of position q of group gid (c / 4 bytes per sub-vector: the lane's N / 2 sub-vectors)
template <int NCW, int N = 32>
__device__ __forceinline__ u32x4 request_codes(const uint8_t* __restrict__ codes, int64_t gid, int q) {
  constexpr int c = CodeBits<NCW>::c;
  const uint8_t* const at = codes + gid * (kGroup / 2 * c / 8) + q * (N / 16 * c);
  const uint32_t* src = reinterpret_cast<const uint32_t*>(at);
  u32x4 out = {0, 0, 0, 0};
  if constexpr (N == 16 && c == 4) {
    out.x = src[0];
  } else if constexpr (N == 16 && c == 6) {            // 6 bytes from a multiple of 6, whose 2-byte part comes last or first
    const bool odd = q & 1;
    const uint32_t w = *reinterpret_cast<const uint32_t*>(at + (odd ? 2 : 0));
    const uint32_t h = *reinterpret_cast<const uint16_t*>(at + (odd ? 0 : 4));
    out.x = odd ? h | (w << 16) : w;
    out.y = odd ? w >> 16 : h;
  } else if constexpr (N == 16) {
    const u32x2 v2 = *reinterpret_cast<const u32x2*>(src);
    out.x = v2.x; out.y = v2.y;
  } else if constexpr (c == 4) {
    const u32x2 v2 = *reinterpret_cast<const u32x2*>(src);
    out.x = v2.x; out.y = v2.y;
  } else if constexpr (c == 6) {
    out.x = src[0]; out.y = src[1]; out.z = src[2];
  } else {
    out = *reinterpret_cast<const u32x4*>(src);
  }
  return out;
}

// the words of position q of head group gid (WIDE: one scale word per token, at gid / 8)
template <int NCW, bool WIDE = false, int N = 32>
__device__ __forceinline__ CodeWords request_words(const uint8_t* __restrict__ codes, const uint16_t* __restrict__ scales,
                                                   int64_t gid, int q) {
  CodeWords w;
  w.code = request_codes<NCW, N>(codes, gid, q);
  if constexpr (is_rtn(NCW)) w.scale = rtn_load_meta<WIDE, N>(scales, gid, q);
  else w.scale = scales[WIDE ? gid >> 3 : gid];
  return w;
}

// Q^-1(codes) + p from the words requested earlier (unrounded, in v); l: group_pos, or with WIDE token_pos
template <int NCW, bool WIDE = false, int N>
__device__ __forceinline__ void dequantize_words(const CodeWords& w, const float (&p)[N], const float (&sf)[N], int l,
                                                 const float4* cb, float (&v)[N]) {
  if constexpr (is_rtn(NCW)) {
    rtn_reconstruct<NCW>(w.code, w.scale, p, v);
  } else {
    uint32_t off[N / 2];
    unpack_offsets<NCW>(w.code, off);
    gather_zhat(off, recon_scale<WIDE>(half_bits_to_float((uint16_t)w.scale), l), cb, v);
    reconstruct<WIDE>(v, l, sf, p);
  }
}

}  // namespace aquakv

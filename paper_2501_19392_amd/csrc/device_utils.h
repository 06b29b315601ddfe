// Device-side helpers shared by the gfx950 streaming kernels: storage-type
// loads/stores, the 128-point Walsh-Hadamard butterfly over a quad of lanes,
// and the reconstruction tail used by quantize / dequantize / scores.
//
// Work decomposition of the streaming kernels: one rotation group (128 values
// of one token and kv head) is held by a QUAD of lanes, 32 consecutive values
// per lane (lane q owns coordinates 32q .. 32q+31).  Five of the seven
// butterfly stages then run inside a lane and only two cross lanes, both as
// DPP quad permutes that fold into the add.  Every global access is a 128-bit
// load/store and the packed codes of a lane are contiguous bytes.
//
// Narrow form (tiles of few rows, whose waves would otherwise leave half of a CU idle): a group is held by EIGHT lanes, 16
// consecutive values each.  The functions below take the lane's values as an array of N = 32 or 16 and do the same operations
// in the same order per value, so both forms give the same bits.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace aquakv {

constexpr int kGroup = 128;          // head_dim = rotation group
constexpr int kLanesPerGroup = 4;
constexpr int kValsPerLane = 32;
constexpr float kRsqrtG = 0.088388347648318440550f;   // 1/sqrt(128)

typedef __bf16 bf16_t;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------- 32-value row access
template <typename T> struct Storage;

// Two-by-two exchange of 16-byte registers between lanes whose positions differ in MASK (1 or 2, inside a quad): the lane without
// that bit keeps a and gets its partner's a for b, the other one keeps b and gets its partner's b for a.  REVERSED: the odd quads
// hold their positions in reverse (token_pos).  One instruction per
// dword: a conditional move whose other side comes through a DPP quad permute.  (Two idle issue slots ahead of a DPP read of a
// register that was just written.)
#define AQUAKV_CND_DPP(out, keep, far, perm) \
  "v_cndmask_b32_dpp %" #out ", %" #far ", %" #keep ", vcc quad_perm:" perm " row_mask:0xf bank_mask:0xf\n\t"
#define AQUAKV_EXCHANGE(perm)                                                                                             \
  "s_mov_b64 vcc, %16\n\ts_nop 1\n\t" AQUAKV_CND_DPP(0, 8, 12, perm) AQUAKV_CND_DPP(1, 9, 13, perm)                      \
  AQUAKV_CND_DPP(2, 10, 14, perm) AQUAKV_CND_DPP(3, 11, 15, perm) "s_not_b64 vcc, vcc\n\t" AQUAKV_CND_DPP(4, 12, 8, perm) \
  AQUAKV_CND_DPP(5, 13, 9, perm) AQUAKV_CND_DPP(6, 14, 10, perm) AQUAKV_CND_DPP(7, 15, 11, perm)
template <int MASK, bool REVERSED> __device__ __forceinline__ void quad_exchange(u32x4& a, u32x4& b) {
  static_assert(MASK == 1 || MASK == 2, "mask");
  const uint64_t without = 0x0101010101010101ull * (MASK == 1 ? (REVERSED ? 0xA5 : 0x55) : (REVERSED ? 0xC3 : 0x33));
  uint32_t o[8];
#define AQUAKV_EXCHANGE_ARGS                                                                                              \
  : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3]), "=&v"(o[4]), "=&v"(o[5]), "=&v"(o[6]), "=&v"(o[7])                  \
  : "v"(a.x), "v"(a.y), "v"(a.z), "v"(a.w), "v"(b.x), "v"(b.y), "v"(b.z), "v"(b.w), "s"(without)                            \
  : "vcc", "scc"
  if constexpr (MASK == 1) asm(AQUAKV_EXCHANGE("[1,0,3,2]") AQUAKV_EXCHANGE_ARGS);
  else asm(AQUAKV_EXCHANGE("[2,3,0,1]") AQUAKV_EXCHANGE_ARGS);
  a = u32x4{o[0], o[1], o[2], o[3]};
  b = u32x4{o[4], o[5], o[6], o[7]};
}

template <> struct Storage<float> {
  template <int N> static __device__ __forceinline__ void load(const float* p, float (&v)[N]) {
#pragma unroll
    for (int c = 0; c < N / 4; ++c) {
      const f32x4 a = reinterpret_cast<const f32x4*>(p)[c];
      v[4 * c] = a.x; v[4 * c + 1] = a.y; v[4 * c + 2] = a.z; v[4 * c + 3] = a.w;
    }
  }
  template <bool REVERSED, int N> static __device__ __forceinline__ void store(float* row, int pos, const float (&v)[N], bool = false) {
    float* const p = row + pos * N;
#pragma unroll
    for (int c = 0; c < N / 4; ++c) {
      f32x4 a;
      a.x = v[4 * c]; a.y = v[4 * c + 1]; a.z = v[4 * c + 2]; a.w = v[4 * c + 3];
      reinterpret_cast<f32x4*>(p)[c] = a;
    }
  }
  static __device__ __forceinline__ float round(float x) { return x; }
};

template <> struct Storage<bf16_t> {
  template <int N> static __device__ __forceinline__ void load(const bf16_t* p, float (&v)[N]) {
#pragma unroll
    for (int c = 0; c < N / 8; ++c) {
      const u32x4 r = reinterpret_cast<const u32x4*>(p)[c];
      const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[8 * c + 2 * i] = __uint_as_float(w[i] << 16);
        v[8 * c + 2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
      }
    }
  }
  static __device__ __forceinline__ uint32_t pack2(float lo, float hi) {
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    f32x2_t f;
    f.x = lo; f.y = hi;
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));   // one packed RNE convert
  }
  // Values N pos ... of a row at p, the lanes of a quad holding consecutive positions.  Lanes that each store their own 64 bytes
  // leave holes between the 16-byte pieces of one instruction, and such stores reach 2.5 TB/s where runs of 64 bytes reach 4.8
  // (32 MiB; 128 MiB: 3.3 against 6.5).  So with 32 values per lane the quad's lanes exchange pieces first, one instruction per
  // value: 64 bytes of a quad per store.  Decode of 32768 tokens 224 -> 212 us, encode 269 / 270 (bound by vector issue).  With 16
  // values, 32 bytes per lane (3.7 and 5.6 TB/s), the exchange costs what it gains.
  // stream (with 32 values per lane): past the L2s (streams()).
  template <bool REVERSED, int N> static __device__ __forceinline__ void store(bf16_t* p, int pos, const float (&v)[N], bool stream = false) {
    constexpr int kPieces = N / 8;
    u32x4 r[kPieces];
#pragma unroll
    for (int c = 0; c < kPieces; ++c) {
      r[c].x = pack2(v[8 * c], v[8 * c + 1]); r[c].y = pack2(v[8 * c + 2], v[8 * c + 3]);
      r[c].z = pack2(v[8 * c + 4], v[8 * c + 5]); r[c].w = pack2(v[8 * c + 6], v[8 * c + 7]);
    }
    if constexpr (kPieces == 4) {
      quad_exchange<1, REVERSED>(r[0], r[1]);
      quad_exchange<1, REVERSED>(r[2], r[3]);
      quad_exchange<2, REVERSED>(r[0], r[2]);
      quad_exchange<2, REVERSED>(r[1], r[3]);
      bf16_t* const at = p + (pos & ~3) * N + (pos & 3) * 8;
#pragma unroll
      for (int c = 0; c < kPieces; ++c) {
        if (stream) {                                     // (the empty statements keep the compiler from making the two stores one)
          asm volatile("");
          __builtin_nontemporal_store(r[c], reinterpret_cast<u32x4*>(at + 32 * c));
          asm volatile("");
        } else {
          *reinterpret_cast<u32x4*>(at + 32 * c) = r[c];
        }
      }
    } else {
#pragma unroll
      for (int c = 0; c < kPieces; ++c) reinterpret_cast<u32x4*>(p + pos * N)[c] = r[c];
    }
  }
  static __device__ __forceinline__ float round(float x) {
    return static_cast<float>(static_cast<bf16_t>(x));
  }
};

// Whether a launch on tiles of 256 rows, or of whole tokens, writes its rows, `elements` bf16 values in all, past the L2s (32 MiB over the
// XCDs): from 16 MiB on its reader, the next launch, finds little of them there, and dirty lines cost their eviction.  A stack of layers, us
// a layer, not / past the L2s: 8192 tokens encode 71.9 / 70.4, decode 54.1 / 55.8, attention 63.9 / 62.6; 38000 tokens 349 / 338, 268 / 264,
// 312 / 306; 131072 (two heads) 1036 / 1030, 807 / 788, 1002 / 984; whole tokens encode 621 / 612 at 65536.  Below 16 MiB the reader is slower: 6200 tokens
// encode 62.0 / 64.3, decode 47.5 / 50.1.  The other tiles never ask: on 320 rows their readers are slower at every size (8300 tokens
// encode 84 / 93, decode 63 / 71, attention 78 / 82; 20000 tokens 182 / 192, 135 / 151, 162 / 172; one layer on three sets of buffers that just fill the 256 MB
// behind the L2s is the exception, decode of 9600 tokens 77 / 70, where 8300 take 64 / 66), and so on 192 rows in several rounds, 32 bytes a
// lane (16500 tokens 158 / 164, 126 / 136, 152 / 154).
__device__ __forceinline__ bool streams(int64_t elements) { return elements >= ((int64_t)1 << 23); }

// 8 bf16 in a 16-byte register quad -> fp32
__device__ __forceinline__ void unpack_bf16x8(const u32x4 r, float* v) {
  const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = __uint_as_float(w[i] << 16);
    v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}

template <int N> __device__ __forceinline__ void load_f32(const float* p, float (&v)[N]) { Storage<float>::load(p, v); }

// ---------------------------------------------------------------- cross-lane moves inside a quad
// Value of `x` held by lane (lane ^ MASK), MASK in {1, 2}: DPP quad_perm.
template <int MASK> __device__ __forceinline__ float quad_xor(float x) {
  static_assert(MASK == 1 || MASK == 2, "mask");
  const int xi = __float_as_int(x);
  constexpr int ctrl = MASK == 1 ? 0xB1 /* [1,0,3,2] */ : 0x4E /* [2,3,0,1] */;
  return __int_as_float(__builtin_amdgcn_mov_dpp(xi, ctrl, 0xF, 0xF, true));   // folds into the consuming add
}

// Sum over the 4 lanes of a group; every lane gets the total (fixed order).
__device__ __forceinline__ float quad_sum(float x) {
  x = x + quad_xor<1>(x);
  x = x + quad_xor<2>(x);
  return x;
}

// ---------------------------------------------------------------- eight lanes per group
// Position (0..7: coordinates 16 pos ... 16 pos + 15) of a lane among the eight of a group.  The upper four lanes hold their
// blocks in reverse, so that the partner whose position differs in bit 2 is lane ^ 7, which a DPP row_half_mirror reads
// (there is no control for lane ^ 4); the positions that differ in bits 0 and 1 are lane ^ 1 and lane ^ 2 as in a quad.
__device__ __forceinline__ int octet_pos(int lane) { return (lane & 7) ^ ((lane & 4) ? 3 : 0); }
__device__ __forceinline__ float octet_mirror(float x) {      // value of lane ^ 7
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x141 /* row_half_mirror */, 0xF, 0xF, true));
}
// Position of `lane` in its group of 4 (N = 32) or 8 (N = 16) lanes.
template <int N> __device__ __forceinline__ int group_pos(int lane) { return N == 32 ? lane & 3 : octet_pos(lane); }

// sum_r a[r] * b[r] over 32 consecutive coordinates as one chain of multiply-adds; with 16 values per lane it passes through two
// lanes, and both get it.
template <int N> __device__ __forceinline__ float chain_dot(const float (&a)[N], const float (&b)[N], int pos) {
  float s = 0.f;
#pragma unroll
  for (int r = 0; r < N; ++r) s = __fmaf_rn(a[r], b[r], s);
  if constexpr (N == 32) return s;
  float t = quad_xor<1>(s);
#pragma unroll
  for (int r = 0; r < N; ++r) t = __fmaf_rn(a[r], b[r], t);
  const float second = quad_xor<1>(t);
  return (pos & 1) ? t : second;
}
// ... over the group, every lane gets it.  Fixed order, the same for both widths: the four chains pairwise.
template <int N> __device__ __forceinline__ float group_dot(const float (&a)[N], const float (&b)[N], int pos) {
  const float s = chain_dot(a, b, pos);
  if constexpr (N == 32) return quad_sum(s);
  const float t = s + quad_xor<2>(s);
  return t + octet_mirror(t);
}

// ---------------------------------------------------------------- 128-point WHT
// v[r] is coordinate 32*q + r of the group (q = lane % 4).  Unnormalised Sylvester-order
// transform: coordinate bits 0..4 are butterflied in registers, bits 5..6 across the quad.
//
// A cross-lane butterfly wants partner + v on the lane holding the 0-bit and partner - v on
// the other.  Both lanes instead run the same multiply-add v + s * partner with a per-lane
// s = +1 / -1 (one DPP instruction per value, exact), which leaves the upper lane with the
// NEGATED result.  The sign is the same for all 32 values of a lane, passes through the
// following (linear) stage unchanged, and is handed back to the caller, who folds it into a
// multiplication it performs anyway:  true transform = quad_sign(q) * (what wht128 leaves in v).
//
// The compiler does not fold the lane permute into a multiply-add, so the stage is written as
// v_fmac_f32 with a DPP quad permute on its first source (dst += permuted(dst) * s).  A DPP
// read of a register written by the VALU instruction just before it needs two idle issue
// slots; the compiler cannot see into the block, so each block of 16 starts with them.  A lane swap (v_permlane16_swap) needs
// them just as well, and the compiler does not count the block's writes: the stage that swaps follow (MASK 8) ends with them too.
#define AQUAKV_FMAC_DPP(i, perm) "v_fmac_f32_dpp %" #i ", %" #i ", %16 " perm " row_mask:0xf bank_mask:0xf\n\t"
#define AQUAKV_FMAC_DPP16(perm)                                                                               \
  "s_nop 1\n\t" AQUAKV_FMAC_DPP(0, perm) AQUAKV_FMAC_DPP(1, perm) AQUAKV_FMAC_DPP(2, perm) AQUAKV_FMAC_DPP(3, perm)  \
  AQUAKV_FMAC_DPP(4, perm) AQUAKV_FMAC_DPP(5, perm) AQUAKV_FMAC_DPP(6, perm) AQUAKV_FMAC_DPP(7, perm)               \
  AQUAKV_FMAC_DPP(8, perm) AQUAKV_FMAC_DPP(9, perm) AQUAKV_FMAC_DPP(10, perm) AQUAKV_FMAC_DPP(11, perm)             \
  AQUAKV_FMAC_DPP(12, perm) AQUAKV_FMAC_DPP(13, perm) AQUAKV_FMAC_DPP(14, perm) AQUAKV_FMAC_DPP(15, perm)
#define AQUAKV_FMAC_ARGS                                                                                              \
  : "+v"(v[b]), "+v"(v[b + 1]), "+v"(v[b + 2]), "+v"(v[b + 3]), "+v"(v[b + 4]), "+v"(v[b + 5]), "+v"(v[b + 6]),        \
    "+v"(v[b + 7]), "+v"(v[b + 8]), "+v"(v[b + 9]), "+v"(v[b + 10]), "+v"(v[b + 11]), "+v"(v[b + 12]),                 \
    "+v"(v[b + 13]), "+v"(v[b + 14]), "+v"(v[b + 15])                                                                  \
  : "v"(s)
// partner lane ^ MASK
template <int MASK, int N> __device__ __forceinline__ void wht_lane_stage(float (&v)[N], float s) {
  static_assert((MASK == 1 || MASK == 2 || MASK == 7 || MASK == 8) && N % 16 == 0, "mask");
#pragma unroll
  for (int b = 0; b < N; b += 16) {
    if constexpr (MASK == 1) asm(AQUAKV_FMAC_DPP16("quad_perm:[1,0,3,2]") AQUAKV_FMAC_ARGS);
    else if constexpr (MASK == 2) asm(AQUAKV_FMAC_DPP16("quad_perm:[2,3,0,1]") AQUAKV_FMAC_ARGS);
    else if constexpr (MASK == 7) asm(AQUAKV_FMAC_DPP16("row_half_mirror") AQUAKV_FMAC_ARGS);
    else asm(AQUAKV_FMAC_DPP16("row_ror:8") "s_nop 1" AQUAKV_FMAC_ARGS);
  }
}

__device__ __forceinline__ float quad_sign(int q) { return (q == 1 || q == 2) ? -1.0f : 1.0f; }

// INV: the inverse-side convention.  The caller has multiplied the lane's INPUT by the parity sign of its lane bits
// (Rot::sign; free when the input is built with a per-lane scale anyway); with s = -1 on the lower and +1 on the upper
// lane of a cross-lane stage, v + s * partner is then the true butterfly on both lanes, (-a) + s (-b) being -(a + s b)
// exactly, and nothing is left pending on the output.
// q: the lane's position in its group (group_pos).
template <bool INV = false, int N> __device__ __forceinline__ void wht128(float (&v)[N], int q) {
  constexpr float up = INV ? 1.0f : -1.0f;               // s on the lane that holds the 1-bit
#pragma unroll
  for (int h = 1; h < N; h <<= 1) {
#pragma unroll
    for (int r = 0; r < N; ++r) {
      if ((r & h) == 0) {
        const float a = v[r], b = v[r + h];
        v[r] = a + b;
        v[r + h] = a - b;
      }
    }
  }
  wht_lane_stage<1>(v, (q & 1) ? up : -up);
  wht_lane_stage<2>(v, (q & 2) ? up : -up);
  if constexpr (N == 16) wht_lane_stage<7>(v, (q & 4) ? up : -up);
}

// ---------------------------------------------------------------- 1024-point WHT (rotation group = whole token)
// A token's 1024 values (8 heads x 128) sit in 1024 / N consecutive lanes, N each: 8 quads, or 8 times eight lanes, that each hold
// one head.  H_1024 = H_8 (x) H_128: after wht128 inside every head, three more butterfly stages pair the positions (token_pos:
// N pos ... are the lane's coordinates) that differ in the three upper bits.  Lanes with bit 2 set hold their blocks in reverse, as
// in octet_pos, so the partners of bits 2 and 3 are lane ^ 7 and lane ^ 8: DPP multiply-adds like the quad stages, with the same
// pending lane sign.  For bits 4 and 5 v_permlane16_swap and v_permlane32_swap bring both values of a butterfly into one lane (they
// exchange the odd rows of 16 lanes, or the upper half of the lanes, of one register with the even rows, or the lower half, of
// another), for two registers at a time, and back: two instructions per value, no pending sign.  (ds_swizzle, which took bits 2
// and 4 before, made a third of the quantizer's LDS instructions.)
template <int N> __device__ __forceinline__ int token_pos(int lane) { return (lane & (1024 / N - 1)) ^ ((lane & 4) ? 3 : 0); }
__device__ __forceinline__ float row_xor8(float x) {     // value of lane ^ 8 (rotation by 8 within a row of 16)
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x128 /* row_ror:8 */, 0xF, 0xF, true));
}
// MASK 16: odd rows of x <-> even rows of y; 32: upper half of x <-> lower half of y
template <int MASK> __device__ __forceinline__ void swap_lanes(float& x, float& y) {
  static_assert(MASK == 16 || MASK == 32, "mask");
  const uint32_t xi = __float_as_uint(x), yi = __float_as_uint(y);
  const auto r = MASK == 16 ? __builtin_amdgcn_permlane16_swap(xi, yi, false, false) : __builtin_amdgcn_permlane32_swap(xi, yi, false, false);
  x = __uint_as_float(r[0]);
  y = __uint_as_float(r[1]);
}
template <int MASK, int N> __device__ __forceinline__ void wht_swap_stage(float (&v)[N]) {
#pragma unroll
  for (int r = 0; r < N / 2; ++r) {
    float a = v[r], b = v[r + N / 2];
    swap_lanes<MASK>(a, b);
    v[r] = a + b;
    v[r + N / 2] = a - b;
    swap_lanes<MASK>(v[r], v[r + N / 2]);
  }
}
template <bool INV = false, int N> __device__ __forceinline__ void wht1024_tail(float (&v)[N], int pos) {
  constexpr float up = INV ? 1.0f : -1.0f;               // as in wht128
  if constexpr (N == 32) wht_lane_stage<7>(v, (pos & 4) ? up : -up);      // (N = 16: bit 2 is a coordinate of the head)
  wht_lane_stage<8>(v, (pos & 8) ? up : -up);
  wht_swap_stage<16>(v);
  if constexpr (N == 16) wht_swap_stage<32>(v);
}
// x of this lane combined with that of the lane whose position differs in bits 4 / 5
template <int MASK> __device__ __forceinline__ float far_sum(float x) {
  float y = x;
  swap_lanes<MASK>(x, y);
  return x + y;
}
// The sum over the lanes of a token of a value that is the same on the lanes of 32 consecutive coordinates; every lane gets the
// total (fixed order, the same for both widths).
template <int N> __device__ __forceinline__ float token_sum(float x) {
  if constexpr (N == 32) x = x + quad_xor<1>(x);
  x = x + quad_xor<2>(x);
  x = x + octet_mirror(x);
  x = x + row_xor8(x);
  x = far_sum<16>(x);
  return N == 16 ? far_sum<32>(x) : x;
}

// Rotation group layouts.  WIDE = false: one group = one head = a quad of lanes (g = 128).  WIDE = true: one group =
// the whole token vector of 8 heads = 1024 / N lanes (g = 1024).  `l` is the lane's position: group_pos, or token_pos.
template <bool WIDE> struct Rot {
  static constexpr float kNorm = WIDE ? 0.03125f : kRsqrtG;            // 1 / sqrt(g)
  static constexpr float kInvG = WIDE ? 1.0f / 1024 : 1.0f / kGroup;
  template <int N> static __device__ __forceinline__ void wht(float (&v)[N], int l) {
    wht128(v, WIDE ? l & (kGroup / N - 1) : l);
    if constexpr (WIDE) wht1024_tail(v, l);
  }
  // The same transform (H_8 (x) H_128 is symmetric) with the stages across the heads first, used for the inverse:
  // a kernel that holds one head of a token per quad and fetches the other heads' grid points itself can then
  // reproduce it bit for bit by adding the 8 heads in the same tree, ((0 1)(2 3))((4 5)(6 7)), before its own wht128.
  // Inverse-side convention (see wht128): input pre-multiplied by sign(l), true output.
  template <int N> static __device__ __forceinline__ void iwht(float (&v)[N], int l) {
    if constexpr (WIDE) wht1024_tail<true>(v, l);
    wht128<true>(v, WIDE ? l & (kGroup / N - 1) : l);
  }
  // sign pending on the lane's values after wht(): -1 for every cross-lane stage in which the lane was the upper one
  // (`l` has one bit per stage; the swapping ones of wht1024_tail leave none)
  static __device__ __forceinline__ float sign(int l) { return (__builtin_popcount(WIDE ? l & 15 : l) & 1) ? -1.0f : 1.0f; }
  // sum of the squares of the group's values
  template <int N> static __device__ __forceinline__ float square_sum(const float (&v)[N], int l) {
    if constexpr (!WIDE) return group_dot(v, v, l);
    return token_sum<N>(chain_dot(v, v, l));
  }
};

// the RHT signs this lane needs as +-1.0f: multiplying by them is exact, so s * x costs one multiplication and
// s * w + p one fused multiply-add that rounds exactly like the addition p +- w
template <int N> __device__ __forceinline__ void load_signs(const int8_t* signs, int head, int q, float (&sf)[N]) {
  const u32x4* src = reinterpret_cast<const u32x4*>(signs + head * kGroup + q * N);
#pragma unroll
  for (int c = 0; c < N / 16; ++c) {
    const u32x4 raw = src[c];
    const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int b = 0; b < 4; ++b)
        sf[16 * c + 4 * i + b] = __uint_as_float(0x3f800000u | (((w[i] >> (8 * b)) & 0x80u) << 24));
  }
}

// Reconstruction: Q^-1(codes) = s * H(sigma16 * C[codes]) / sqrt(g).  The transform is linear, so the factor
// 1 / sqrt(g) goes into the scale once per group, together with the lane's parity sign that the inverse-side
// convention of the cross-lane stages wants on its input: the grid points are multiplied by recon_scale(sigma16, l)
// when they are fetched, and after the inverse transform one fused multiply-add per value applies the RHT sign and
// adds the prediction.  Used unchanged by the quantize,
// dequantize, scoring and fused kernels so that all of them produce bit-identical keys / values.
template <bool WIDE = false> __device__ __forceinline__ float recon_scale(float s16, int l) {
  return s16 * (Rot<WIDE>::sign(l) * Rot<WIDE>::kNorm);
}
// z: grid points scaled by recon_scale (rotated domain) -> p + Q^-1(codes)
template <bool WIDE = false, int N>
__device__ __forceinline__ void reconstruct(float (&z)[N], int l, const float (&sf)[N], const float (&p)[N]) {
  Rot<WIDE>::iwht(z, l);
#pragma unroll
  for (int r = 0; r < N; ++r) z[r] = __fmaf_rn(z[r], sf[r], p[r]);
}

// Rotary embedding (RoFormer) of the coordinates this lane holds of a 128-long head vector.  Coordinate d is
// paired with d + 64, which is the same register of the lane whose position differs in the uppermost bit; `cos_t` / `sin_t`
// point at the 64 angles of the token's position.  x'_d = x_d cos - x_{d+64} sin,  x'_{d+64} = x_{d+64} cos + x_d sin.
template <int N>
__device__ __forceinline__ void rope128(float (&v)[N], int q, const float* __restrict__ cos_t,
                                        const float* __restrict__ sin_t) {
  constexpr int kUpper = 64 / N;                         // the position's uppermost bit
  float c[N], s[N];
  load_f32(cos_t + N * (q & (kUpper - 1)), c);
  load_f32(sin_t + N * (q & (kUpper - 1)), s);
  const float sgn = (q & kUpper) ? 1.0f : -1.0f;
#pragma unroll
  for (int r = 0; r < N; ++r) {
    float partner;
    if constexpr (N == 32) partner = quad_xor<2>(v[r]);
    else partner = octet_mirror(v[r]);
    v[r] = __fmaf_rn(v[r], c[r], sgn * (partner * s[r]));
  }
}

}  // namespace aquakv

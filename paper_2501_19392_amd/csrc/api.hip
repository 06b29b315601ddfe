// C-ABI layer: argument validation, workspace layout, chunking and dispatch.
// No HIP call is made before validation has passed.
#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <memory>
#include <mutex>
#include <new>

#include "../../include/aquakv.h"
#include "kernels.h"

namespace {

thread_local char g_err[512] = "";

int fail(int status, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return status;
}

// Rows handled per pass of the layer-level calls.  bf16 layers run the fused kernels, which
// need no prediction buffer (the chunk only bounds the temporary Khat).  fp32 layers run
// predictor and quantizer as separate kernels: the fp32 predictions of one chunk
// (chunk * D * 4 bytes) then stay close to the caches between the two.
constexpr int64_t kChunkRowsFused = 65536;
constexpr int64_t kChunkRowsSplit = 16384;

inline bool misaligned(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }
inline size_t elem_bytes(int dtype) { return dtype == AQUAKV_BF16 ? 2 : 4; }
// Sect. 4.1 "Backbone quantization": vq_dim 2 = grid in R^2 behind a Hadamard rotation, vq_dim 1 = uniform
// round-to-nearest on groups of 64 channels
inline bool is_rtn(const aquakv_layer* L) { return L->vq_dim == 1; }
constexpr int kRtnGroup = 64;
// what the kernels are instantiated on: the grid size, or the bits per value of the round-to-nearest backbone
inline int quantizer_id(const aquakv_layer* L) { return is_rtn(L) ? (L->n_codewords == 4 ? 2 : 4) : L->n_codewords; }
// code bits per pair of values
inline int code_bits(const aquakv_layer* L) {
  if (is_rtn(L)) return L->n_codewords == 4 ? 4 : 8;
  return L->n_codewords == 16 ? 4 : L->n_codewords == 64 ? 6 : 8;
}

int check_layer(const aquakv_layer* L) {
  if (L == nullptr) return fail(AQUAKV_ENULL, "layer is NULL");
  if (L->kv_heads < 1 || L->kv_heads > 4096) return fail(AQUAKV_EINVAL, "kv_heads=%d out of range", L->kv_heads);
  if (L->head_dim < 1 || (L->head_dim & (L->head_dim - 1)))
    return fail(AQUAKV_EINVAL, "head_dim=%d is not a power of two", L->head_dim);
  if (L->head_dim != 128) return fail(AQUAKV_EUNSUPPORTED, "head_dim=%d: only 128 is built", L->head_dim);
  if (L->vq_dim < 1) return fail(AQUAKV_EINVAL, "vq_dim=%d", L->vq_dim);
  if (L->vq_dim > 2) return fail(AQUAKV_EUNSUPPORTED, "vq_dim=%d: only 1 and 2 are built", L->vq_dim);
  const bool pow2 = L->n_codewords >= 2 && !(L->n_codewords & (L->n_codewords - 1));
  if (is_rtn(L)) {
    if (L->n_codewords != 4 && L->n_codewords != 16)
      return fail(pow2 ? AQUAKV_EUNSUPPORTED : AQUAKV_EINVAL, "n_codewords=%d: vq_dim 1 is built for 4 or 16 levels", L->n_codewords);
    if (L->rht_group != 0 && L->rht_group != kRtnGroup && !(L->rht_group == 1024 && L->kv_heads * L->head_dim == 1024))
      return fail(AQUAKV_EUNSUPPORTED, "rht_group=%d: vq_dim 1 is built for groups of %d, and of 1024 = the whole token of 8 heads",
                  L->rht_group, kRtnGroup);
  } else if (L->n_codewords != 16 && L->n_codewords != 64 && L->n_codewords != 256) {
    return fail(pow2 ? AQUAKV_EUNSUPPORTED : AQUAKV_EINVAL, "n_codewords=%d: must be 16, 64 or 256", L->n_codewords);
  }
  if (L->dtype != AQUAKV_BF16 && L->dtype != AQUAKV_FP32) return fail(AQUAKV_EINVAL, "dtype=%d", L->dtype);
  const int D = L->kv_heads * L->head_dim;
  if (!is_rtn(L) && L->rht_group != 0 && L->rht_group != L->head_dim) {
    if (L->rht_group != D) return fail(AQUAKV_EINVAL, "rht_group=%d must be 0, head_dim or kv_heads * head_dim", L->rht_group);
    if (D != 1024) return fail(AQUAKV_EUNSUPPORTED, "rht_group=%d: groups across heads are built for 8 heads of 128", L->rht_group);
  }
  if (L->d_in_k < 0 || L->d_in_k % 128) return fail(AQUAKV_EINVAL, "d_in_k=%d must be a non-negative multiple of 128", L->d_in_k);
  if (L->d_in_v < 0 || L->d_in_v % 128) return fail(AQUAKV_EINVAL, "d_in_v=%d must be a non-negative multiple of 128", L->d_in_v);
  if (L->d_in_v != 0 && L->d_in_v <= D)
    return fail(AQUAKV_EINVAL, "d_in_v=%d must exceed D=%d (inputs are [Vhat_prev | Khat])", L->d_in_v, D);
  if (!is_rtn(L)) {      // the round-to-nearest backbone has neither grid nor rotation; the three pointers are ignored
    if (L->codebook == nullptr) return fail(AQUAKV_ENULL, "codebook is NULL");
    if (L->signs_k == nullptr || L->signs_v == nullptr) return fail(AQUAKV_ENULL, "signs_k / signs_v is NULL");
  }
  if (L->d_in_k && L->w_k == nullptr) return fail(AQUAKV_ENULL, "w_k is NULL but d_in_k=%d", L->d_in_k);
  if (L->d_in_v && L->w_v == nullptr) return fail(AQUAKV_ENULL, "w_v is NULL but d_in_v=%d", L->d_in_v);
  const void* used[] = {L->w_k, L->b_k, L->w_v, L->b_v};
  for (const void* p : used)
    if (p != nullptr && misaligned(p)) return fail(AQUAKV_EALIGN, "a pointer in aquakv_layer is not 16-byte aligned");
  if (!is_rtn(L)) {      // ignored (never read, whatever they hold) by the round-to-nearest backbone
    const void* grid[] = {L->codebook, L->signs_k, L->signs_v, L->search_table};
    for (const void* p : grid)
      if (p != nullptr && misaligned(p)) return fail(AQUAKV_EALIGN, "a pointer in aquakv_layer is not 16-byte aligned");
  }
  return AQUAKV_OK;
}

// rotation group = the whole token vector (Sect. 4.1 of the paper) instead of one head
inline bool is_wide(const aquakv_layer* L) {
  if (is_rtn(L)) return L->rht_group == 1024;
  return L->rht_group != 0 && L->rht_group != L->head_dim;
}
// bytes of scales per token row: one fp16 per rotation group, or (fp16 step, 16-bit zero point) per group of 64
inline size_t scale_row_bytes(const aquakv_layer* L) {
  if (is_rtn(L)) return (is_wide(L) ? 1 : (size_t)L->kv_heads * (L->head_dim / kRtnGroup)) * 2 * sizeof(uint16_t);
  return (is_wide(L) ? 1 : (size_t)L->kv_heads) * sizeof(uint16_t);
}

int check_ptr(const void* p, const char* name, bool required) {
  if (p == nullptr) return required ? fail(AQUAKV_ENULL, "%s is NULL", name) : AQUAKV_OK;
  if (misaligned(p)) return fail(AQUAKV_EALIGN, "%s is not 16-byte aligned", name);
  return AQUAKV_OK;
}

// scales are read and written one fp16 at a time: with one scale per token a row range of the cache starts at
// any even address
// (the round-to-nearest backbone stores a step and a zero point together as one 4-byte word)
int check_scales(const aquakv_layer* L, const void* p, const char* name, bool required) {
  if (p == nullptr) return required ? fail(AQUAKV_ENULL, "%s is NULL", name) : AQUAKV_OK;
  const unsigned need = is_rtn(L) ? 4u : 2u;
  if (reinterpret_cast<uintptr_t>(p) & (need - 1u)) return fail(AQUAKV_EALIGN, "%s is not %u-byte aligned", name, need);
  return AQUAKV_OK;
}

// Byte ranges [p, p + n) of the buffers of one call.  The kernels of a call read whole rows of their inputs
// while other workgroups write outputs for the same rows, so an output that overlaps an input it may not
// alias (or another output, or the workspace) is a race; it is refused before anything is launched.
struct Range { const void* p; size_t n; const char* name; };
inline bool overlap(const Range& a, const Range& b) {
  if (a.p == nullptr || b.p == nullptr || a.n == 0 || b.n == 0) return false;
  const uintptr_t a0 = reinterpret_cast<uintptr_t>(a.p), b0 = reinterpret_cast<uintptr_t>(b.p);
  return a0 < b0 + b.n && b0 < a0 + a.n;
}
// every output against every input and against the other outputs; `inplace` (nullable, one entry per output)
// names the one input an output may coincide with exactly (reconstruction in place)
int check_no_alias(const Range* outs, int n_out, const Range* ins, int n_in, const void* const* inplace = nullptr) {
  for (int i = 0; i < n_out; ++i) {
    for (int j = 0; j < n_in; ++j) {
      if (inplace != nullptr && inplace[i] != nullptr && inplace[i] == ins[j].p && outs[i].p == ins[j].p) continue;
      if (overlap(outs[i], ins[j])) return fail(AQUAKV_EINVAL, "%s overlaps %s", outs[i].name, ins[j].name);
    }
    for (int j = i + 1; j < n_out; ++j)
      if (overlap(outs[i], outs[j])) return fail(AQUAKV_EINVAL, "%s overlaps %s", outs[i].name, outs[j].name);
  }
  return AQUAKV_OK;
}

// The same over the many buffers of a call on a whole cache: no buffer that is written may overlap any other one (`shared`: but those
// written may overlap one another).  In order of address, a range overlaps an earlier one iff it starts before the furthest end so far,
// of any range (shared: of those read) if it is written itself, else of the written ones.
struct CacheRange { uintptr_t begin, end; const char* name; int32_t layer; bool written; };
int check_disjoint(CacheRange* r, int64_t n, bool shared = false) {
  std::sort(r, r + n, [](const CacheRange& a, const CacheRange& b) { return a.begin < b.begin; });
  const CacheRange *read = nullptr, *written = nullptr;     // the ones that reach furthest
  for (int64_t i = 0; i < n; ++i) {
    for (const CacheRange* before : {r[i].written ? read : nullptr, r[i].written && shared ? nullptr : written})
      if (before != nullptr && r[i].begin < before->end)
        return fail(AQUAKV_EINVAL, "%s of layer %d overlaps %s of layer %d", r[i].name, r[i].layer, before->name, before->layer);
    const CacheRange*& furthest = r[i].written ? written : read;
    if (furthest == nullptr || r[i].end > furthest->end) furthest = r + i;
  }
  return AQUAKV_OK;
}

#define CHECK(expr)                      \
  do {                                   \
    const int s_ = (expr);               \
    if (s_ != AQUAKV_OK) return s_;      \
  } while (0)

#define HIP_TRY(expr)                                                                     \
  do {                                                                                    \
    const hipError_t e_ = (expr);                                                         \
    if (e_ != hipSuccess) return fail(AQUAKV_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

struct Plan {
  int D;
  size_t eb;          // bytes per element of the storage dtype
  size_t code_row;    // bytes of codes per token row
  int64_t chunk;      // rows per pass
  bool fused;         // bf16: predictor fused with the quantizer kernels
  bool fused_dec;     // bf16: predictor fused with the inverse quantizer (also for groups across the 8 heads)
  size_t p_bytes;     // front of the workspace: fp32 predictions of one chunk, or re-tiled predictor weights
  size_t khat_bytes;  // temporary Khat of one chunk
};

Plan make_plan(const aquakv_layer* L, int64_t tokens) {
  Plan pl;
  pl.D = L->kv_heads * L->head_dim;
  pl.eb = elem_bytes(L->dtype);
  pl.code_row = (size_t)L->kv_heads * (L->head_dim / 2) * code_bits(L) / 8;
  pl.fused = L->dtype == AQUAKV_BF16;                  // predictor fused with the quantizer (groups of one head: a tile of one
                                                       // head; groups across the 8 heads: a slab of 64 tokens x all heads)
  pl.fused_dec = L->dtype == AQUAKV_BF16;              // decoding needs no statistic of the whole group
  const int64_t cap = pl.fused ? kChunkRowsFused : kChunkRowsSplit;
  pl.chunk = tokens < cap ? tokens : cap;
  // front of the workspace: the fp32 predictions of a chunk (split path), or (bf16, groups across the heads) the
  // predictor weights re-tiled for the encoder's main loop
  const int d_in_max = L->d_in_k > L->d_in_v ? L->d_in_k : L->d_in_v;
  pl.p_bytes = !pl.fused ? (size_t)pl.chunk * pl.D * sizeof(float) : (is_wide(L) ? (size_t)pl.D * d_in_max * pl.eb : 0);
  pl.khat_bytes = (size_t)pl.chunk * pl.D * pl.eb;
  return pl;
}

// Encode of rotation groups across the 8 heads (encode_wide): rows that the kernel of whole tokens takes in one round over the
// CUs, and up to how many left over from its rounds may be quantized from fp32 predictions (wide_split_rows).
constexpr int64_t kWideRoundRows = 16384, kWideSplitRows = 12288;

// The parameters that calls on a layer read.
struct Params { Range r[8]; };
Params params_of(const aquakv_layer* L) {
  const size_t D = (size_t)L->kv_heads * L->head_dim, eb = elem_bytes(L->dtype), points = is_rtn(L) ? 0 : (size_t)L->n_codewords;
  return {{{L->w_k, D * L->d_in_k * eb, "w_k"}, {L->w_v, D * L->d_in_v * eb, "w_v"},
           {L->b_k, L->d_in_k ? D * sizeof(float) : 0, "b_k"}, {L->b_v, L->d_in_v ? D * sizeof(float) : 0, "b_v"},
           {L->signs_k, points ? D : 0, "signs_k"}, {L->signs_v, points ? D : 0, "signs_v"},
           {L->codebook, points * 2 * sizeof(float), "codebook"},
           {L->search_table, points ? aquakv::kSearchTableBytes : 0, "search_table"}}};
}

// Whether `all` lies over none of the call's buffers (outs: without the workspace it is part of) nor the layer's parameters.
bool clear_of(const aquakv_layer* L, const Range& all, const Range* outs, int n_out, const Range* ins, int n_in) {
  for (const Range& r : params_of(L).r)
    if (overlap(all, r)) return false;
  for (int i = 0; i < n_out; ++i)
    if (overlap(all, outs[i])) return false;
  for (int j = 0; j < n_in; ++j)
    if (overlap(all, ins[j])) return false;
  return true;
}

// Bytes of the workspace an encode call over `tokens` rows uses: the `sure` bytes it cannot do without, the `need` bytes every caller
// provides (the room of a temporary Khat holds predictions where there is a Khat to write to), and where more predictions help up to as
// much as those of all rows take.  What lies behind the first `sure` bytes is left alone if any of it is over the call's other
// buffers or the layer's parameters: an arena's owner may state all that is left of it.
size_t usable_workspace(const aquakv_layer* L, const Plan& pl, int64_t tokens, void* workspace, size_t sure, size_t need, size_t bytes,
                        const Range* outs, int n_out, const Range* ins, int n_in) {
  if (!pl.fused || !is_wide(L) || (L->d_in_k == 0 && L->d_in_v == 0)) return sure;
  const size_t all = need + (size_t)tokens * pl.D * sizeof(float);
  const size_t most = tokens > kWideSplitRows ? need : bytes < all ? bytes : all;
  for (const size_t n : {most, need})
    if (n > sure && clear_of(L, {workspace, n, ""}, outs, n_out, ins, n_in)) return n;
  return sure;
}
// Keys and values of `tokens` rows can run as launch_fused_layer, given room for half of its sums and, in Vhat, for the other half.
inline bool layer_at_once(const aquakv_layer* L, const Plan& pl, int64_t tokens, const void* V, const void* Vhat) {
  return pl.fused && L->d_in_k != 0 && L->d_in_v != 0 && Vhat != nullptr && Vhat != V && aquakv::fused_layer_fits(tokens, pl.D);
}

inline const void* at(const void* base, int64_t row, size_t row_bytes) {
  return base == nullptr ? nullptr : static_cast<const unsigned char*>(base) + row * row_bytes;
}
inline void* at(void* base, int64_t row, size_t row_bytes) {
  return base == nullptr ? nullptr : static_cast<unsigned char*>(base) + row * row_bytes;
}

// a tensor to be recovered from its codes
inline aquakv::QuantizeIo coded(const int8_t* signs, const void* codes, const void* scales, void* hat) {
  return {nullptr, signs, static_cast<uint8_t*>(const_cast<void*>(codes)), static_cast<uint16_t*>(const_cast<void*>(scales)), hat};
}

// Up to how many rows predictions in `pieces` pieces are cheaper than another round of whole tokens; `ahead`: behind such rounds, where
// inputs and predictions of a large range come from memory.  Every piece starts both launches anew, and the round costs more the
// more points there are to search (uniform backbone: none).  Keys and values, us, predictions / whole tokens.  One piece: 16 points 4096 rows
// 74 / 152, 8192 115 / 153, 12288 139 / 156, 13000 155 / 158 (uniform 60 / 111, 97 / 111, 117 / 117, 129 / 119); behind a round, with it,
// 4096 rows 258 / 314, 9000 316 / 323, 12288 327 / 326 (uniform 201 / 234, 261 / 245, 273 / 251).  Two pieces of both tensors (in place):
// 8192 138 / 145 (uniform 116 / 113, 7000: 110 / 112), 9000 199 / 144; behind a round (no Khat) 4096 289 / 315.  Three: 6000 147 / 153
// (uniform 119 / 112), behind a round 336 / 317 (256 points 419 / 439).  Four: 7000 187 / 153; of the values alone 4096 130 / 146, behind a
// round 299 / 290 (256 points 383 / 418).
inline int64_t wide_split_rows(const aquakv_layer* L, bool ahead, int64_t pieces) {
  constexpr int64_t rows[3][2][4] = {{{kWideSplitRows, 8192, 6144, 4096}, {kWideSplitRows, 4096, 3072, 0}},
                                     {{kWideSplitRows, 8192, 6144, 4096}, {kWideSplitRows, 6144, 6144, 4096}},      // 256 points
                                     {{kWideSplitRows, 7168, 4096, 4096}, {4096, 4096, 3072, 0}}};                  // uniform
  return pieces < 1 || pieces > 4 ? 0 : rows[is_rtn(L) ? 2 : L->n_codewords == 256][ahead][pieces - 1];
}

// Encode of n rows of one tensor with rotation groups across the 8 heads.  The kernel that owns whole tokens walks all of W in
// every workgroup of 64 tokens, so a round of it over the CUs costs the same however few of them it fills.  It takes whole rounds;
// what is left over runs as predictor and stand-alone quantizer if that is cheaper than another round (wide_split_rows): predictions in
// fp32, half of each row in the workspace (`room` bytes) and half in the row of Xhat that comes to lie over it, or, without an Xhat of its
// own, all of it in the workspace; in pieces of as many rows as there is room for.
int encode_wide(const aquakv_layer* L, const void* x0, int d0, const void* x1, int d1, const void* W, const float* bias,
                const int8_t* signs, const void* X, uint8_t* codes, uint16_t* scales, void* Xhat, int64_t n, int D, float* ws,
                size_t room, hipStream_t stream) {
  const size_t eb = elem_bytes(L->dtype), row = (size_t)D * eb;
  const int64_t rest = n % kWideRoundRows;
  const bool halves = Xhat != nullptr && Xhat != X;
  const int64_t fit = (int64_t)(room / (halves ? row : (size_t)D * sizeof(float)));
  const int64_t pieces = fit > 0 ? (rest + fit - 1) / fit : 0, piece = pieces > 0 ? (rest + pieces - 1) / pieces : 0;
  const int64_t whole = rest > wide_split_rows(L, n != rest, pieces) ? n : n - rest;
  if (whole != 0)
    HIP_TRY(aquakv::launch_fused_encode_wide(quantizer_id(L), x0, d0, x1, d1, W, ws, bias, signs, L->codebook, L->search_table, X,
                                             codes, scales, Xhat, whole, D, stream));
  for (int64_t r = whole; r < n; r += piece) {
    const int64_t m = n - r < piece ? n - r : piece;
    const aquakv::Prediction P = halves ? aquakv::Prediction{static_cast<float*>(at(Xhat, r, row)), ws, D / 2, D / 2}
                                        : aquakv::Prediction::contiguous(ws, D);
    HIP_TRY(aquakv::launch_tile_predict(at(x0, r, d0 * eb), d0, at(x1, r, d1 * eb), d1, W, bias, P, m, D, stream));
    const aquakv::QuantizeIo io = {at(X, r, row), signs, codes + r * (int64_t)(D / 2 * code_bits(L) / 8),
                                   static_cast<uint16_t*>(at(scales, r, scale_row_bytes(L))), at(Xhat, r, row)};
    HIP_TRY(aquakv::launch_quantize(L->dtype, quantizer_id(L), &io, 1, &P, L->codebook, L->search_table, m, L->kv_heads, true, stream));
  }
  return AQUAKV_OK;
}

// ---- one chunk of rows [r0, r0 + n) of one tensor; pointers are the tensors' bases -------------------------------
// keys of Alg. "encode":  K_pred = f_key(Khat_prev);  K_q = Q(K - K_pred);  khat_dst (chunk-local, nullable) = Q^-1(K_q) + K_pred
int encode_keys_chunk(const aquakv_layer* L, const Plan& pl, int64_t r0, int64_t n, const void* K, const void* Khat_prev,
                      uint8_t* k_codes, uint16_t* k_scales, void* khat_dst, float* Pbuf, size_t room, hipStream_t stream) {
  const bool has_k = L->d_in_k != 0;
  const size_t row = (size_t)pl.D * pl.eb, srow = scale_row_bytes(L);
  if (has_k && pl.fused) {
    const void* x0 = at(Khat_prev, r0, (size_t)L->d_in_k * pl.eb);
    uint8_t* const kc = static_cast<uint8_t*>(at(k_codes, r0, pl.code_row));
    uint16_t* const ks = static_cast<uint16_t*>(at(k_scales, r0, srow));
    if (is_wide(L))
      return encode_wide(L, x0, L->d_in_k, nullptr, 0, L->w_k, L->b_k, L->signs_k, at(K, r0, row), kc, ks, khat_dst, n, pl.D, Pbuf,
                         room, stream);
    HIP_TRY(aquakv::launch_fused_encode(quantizer_id(L), x0, L->d_in_k, nullptr, 0, L->w_k, L->b_k, L->signs_k, L->codebook,
                                        L->search_table, at(K, r0, row), kc, ks, khat_dst, n, pl.D, stream));
    return AQUAKV_OK;
  }
  if (has_k)
    HIP_TRY(aquakv::launch_predict(L->dtype, at(Khat_prev, r0, (size_t)L->d_in_k * pl.eb), L->d_in_k, nullptr, 0, L->w_k,
                                   L->b_k, Pbuf, n, pl.D, stream));
  const aquakv::QuantizeIo io = {at(K, r0, row), L->signs_k, static_cast<uint8_t*>(at(k_codes, r0, pl.code_row)),
                                 static_cast<uint16_t*>(at(k_scales, r0, srow)), khat_dst};
  const aquakv::Prediction P = aquakv::Prediction::contiguous(Pbuf, pl.D);
  HIP_TRY(aquakv::launch_quantize(L->dtype, quantizer_id(L), &io, 1, has_k ? &P : nullptr, L->codebook, L->search_table, n,
                                  L->kv_heads, is_wide(L), stream));
  return AQUAKV_OK;
}

// values of Alg. "encode":  V_pred = f_value([Vhat_prev; Khat]);  V_q = Q(V - V_pred);  khat_src is chunk-local
int encode_values_chunk(const aquakv_layer* L, const Plan& pl, int64_t r0, int64_t n, const void* V, const void* Vhat_prev,
                        const void* khat_src, uint8_t* v_codes, uint16_t* v_scales, void* Vhat, float* Pbuf,
                        size_t room, hipStream_t stream) {
  const bool has_v = L->d_in_v != 0;
  const int D = pl.D;
  const size_t row = (size_t)D * pl.eb, srow = scale_row_bytes(L);
  if (has_v && pl.fused) {
    const void* x0 = at(Vhat_prev, r0, (size_t)(L->d_in_v - D) * pl.eb);
    uint8_t* const vc = static_cast<uint8_t*>(at(v_codes, r0, pl.code_row));
    uint16_t* const vs = static_cast<uint16_t*>(at(v_scales, r0, srow));
    if (is_wide(L))
      return encode_wide(L, x0, L->d_in_v - D, khat_src, D, L->w_v, L->b_v, L->signs_v, at(V, r0, row), vc, vs, at(Vhat, r0, row),
                         n, D, Pbuf, room, stream);
    HIP_TRY(aquakv::launch_fused_encode(quantizer_id(L), x0, L->d_in_v - D, khat_src, D, L->w_v, L->b_v, L->signs_v,
                                        L->codebook, L->search_table, at(V, r0, row), vc, vs, at(Vhat, r0, row), n, D, stream));
    return AQUAKV_OK;
  }
  if (has_v)
    HIP_TRY(aquakv::launch_predict(L->dtype, at(Vhat_prev, r0, (size_t)(L->d_in_v - D) * pl.eb), L->d_in_v - D, khat_src, D,
                                   L->w_v, L->b_v, Pbuf, n, D, stream));
  const aquakv::QuantizeIo io = {at(V, r0, row), L->signs_v, static_cast<uint8_t*>(at(v_codes, r0, pl.code_row)),
                                 static_cast<uint16_t*>(at(v_scales, r0, srow)), at(Vhat, r0, row)};
  const aquakv::Prediction P = aquakv::Prediction::contiguous(Pbuf, D);
  HIP_TRY(aquakv::launch_quantize(L->dtype, quantizer_id(L), &io, 1, has_v ? &P : nullptr, L->codebook, L->search_table, n,
                                  L->kv_heads, is_wide(L), stream));
  return AQUAKV_OK;
}

// keys of Alg. "decode":  Khat = Q^-1(K_q) + f_key(Khat_prev)
int decode_keys_chunk(const aquakv_layer* L, const Plan& pl, int64_t r0, int64_t n, const uint8_t* k_codes,
                      const uint16_t* k_scales, const void* Khat_prev, void* Khat, float* Pbuf, hipStream_t stream) {
  const bool has_k = L->d_in_k != 0;
  const size_t row = (size_t)pl.D * pl.eb, srow = scale_row_bytes(L);
  if (has_k && pl.fused_dec) {
    HIP_TRY(aquakv::launch_fused_decode(quantizer_id(L), at(Khat_prev, r0, (size_t)L->d_in_k * pl.eb), L->d_in_k, nullptr, 0,
                                        L->w_k, L->b_k, L->signs_k, L->codebook,
                                        static_cast<const uint8_t*>(at(k_codes, r0, pl.code_row)),
                                        static_cast<const uint16_t*>(at(k_scales, r0, srow)), at(Khat, r0, row), n, pl.D,
                                        is_wide(L), stream));
    return AQUAKV_OK;
  }
  if (has_k)
    HIP_TRY(aquakv::launch_predict(L->dtype, at(Khat_prev, r0, (size_t)L->d_in_k * pl.eb), L->d_in_k, nullptr, 0, L->w_k,
                                   L->b_k, Pbuf, n, pl.D, stream));
  const aquakv::QuantizeIo io = coded(L->signs_k, at(k_codes, r0, pl.code_row), at(k_scales, r0, srow), at(Khat, r0, row));
  HIP_TRY(aquakv::launch_dequantize(L->dtype, quantizer_id(L), &io, 1, has_k ? Pbuf : nullptr, L->codebook, n, L->kv_heads,
                                    is_wide(L), stream));
  return AQUAKV_OK;
}

// values of Alg. "decode":  Vhat = Q^-1(V_q) + f_value([Vhat_prev; Khat])
int decode_values_chunk(const aquakv_layer* L, const Plan& pl, int64_t r0, int64_t n, const uint8_t* v_codes,
                        const uint16_t* v_scales, const void* Vhat_prev, const void* Khat, void* Vhat, float* Pbuf,
                        hipStream_t stream) {
  const bool has_v = L->d_in_v != 0;
  const int D = pl.D;
  const size_t row = (size_t)D * pl.eb, srow = scale_row_bytes(L);
  if (has_v && pl.fused_dec) {
    HIP_TRY(aquakv::launch_fused_decode(quantizer_id(L), at(Vhat_prev, r0, (size_t)(L->d_in_v - D) * pl.eb), L->d_in_v - D,
                                        at(Khat, r0, row), D, L->w_v, L->b_v, L->signs_v, L->codebook,
                                        static_cast<const uint8_t*>(at(v_codes, r0, pl.code_row)),
                                        static_cast<const uint16_t*>(at(v_scales, r0, srow)), at(Vhat, r0, row), n, D,
                                        is_wide(L), stream));
    return AQUAKV_OK;
  }
  if (has_v)
    HIP_TRY(aquakv::launch_predict(L->dtype, at(Vhat_prev, r0, (size_t)(L->d_in_v - D) * pl.eb), L->d_in_v - D,
                                   at(Khat, r0, row), D, L->w_v, L->b_v, Pbuf, n, D, stream));
  const aquakv::QuantizeIo io = coded(L->signs_v, at(v_codes, r0, pl.code_row), at(v_scales, r0, srow), at(Vhat, r0, row));
  HIP_TRY(aquakv::launch_dequantize(L->dtype, quantizer_id(L), &io, 1, has_v ? Pbuf : nullptr, L->codebook, n, L->kv_heads,
                                    is_wide(L), stream));
  return AQUAKV_OK;
}

}  // namespace

extern "C" {

int aquakv_version(void) { return AQUAKV_VERSION; }

const char* aquakv_status_string(int status) {
  switch (status) {
    case AQUAKV_OK: return "ok";
    case AQUAKV_EINVAL: return "invalid argument";
    case AQUAKV_ENULL: return "required pointer is NULL";
    case AQUAKV_EALIGN: return "pointer is not 16-byte aligned";
    case AQUAKV_EUNSUPPORTED: return "configuration not built";
    case AQUAKV_EWORKSPACE: return "workspace too small";
    case AQUAKV_EHIP: return "HIP error";
    default: return "unknown status";
  }
}

const char* aquakv_last_error(void) { return g_err; }

size_t aquakv_search_table_bytes(int32_t n_codewords) {
  return (n_codewords == 16 || n_codewords == 64 || n_codewords == 256) ? aquakv::kSearchTableBytes : 0;
}

int aquakv_build_search_table(const float* codebook, int32_t vq_dim, int32_t n_codewords, void* table, void* stream) {
  if (vq_dim != 2) return fail(vq_dim < 1 ? AQUAKV_EINVAL : AQUAKV_EUNSUPPORTED, "vq_dim=%d: only 2 is built", vq_dim);
  if (aquakv_search_table_bytes(n_codewords) == 0)
    return fail(AQUAKV_EINVAL, "n_codewords=%d: must be 16, 64 or 256", n_codewords);
  CHECK(check_ptr(codebook, "codebook", true));
  CHECK(check_ptr(table, "table", true));
  HIP_TRY(aquakv::launch_build_search_table(codebook, n_codewords, table, static_cast<hipStream_t>(stream)));
  return AQUAKV_OK;
}

size_t aquakv_workspace_bytes(const aquakv_layer* layer, int64_t tokens) {
  if (check_layer(layer) != AQUAKV_OK || tokens <= 0) return 0;
  const Plan pl = make_plan(layer, tokens);
  return pl.p_bytes + pl.khat_bytes;
}

int aquakv_fused_tile_heads(const aquakv_layer* layer, int64_t tokens) {
  if (check_layer(layer) != AQUAKV_OK || tokens <= 0) return 0;
  const Plan pl = make_plan(layer, tokens);
  if (!pl.fused_dec || layer->d_in_k == 0) return 0;
  return aquakv::two_heads_pays(pl.chunk, pl.D) ? 2 : 1;
}

int aquakv_predict(const aquakv_layer* L, int which, int64_t tokens, const void* x0, const void* x1, float* P,
                   void* stream) {
  CHECK(check_layer(L));
  if (which != AQUAKV_KEY && which != AQUAKV_VALUE) return fail(AQUAKV_EINVAL, "which=%d", which);
  if (tokens < 0) return fail(AQUAKV_EINVAL, "tokens=%lld", (long long)tokens);
  const int D = L->kv_heads * L->head_dim;
  const int d_in = which == AQUAKV_KEY ? L->d_in_k : L->d_in_v;
  if (d_in == 0) return fail(AQUAKV_EINVAL, "the layer has no %s predictor", which == AQUAKV_KEY ? "key" : "value");
  CHECK(check_ptr(x0, "x0", true));
  CHECK(check_ptr(x1, "x1", which == AQUAKV_VALUE));
  CHECK(check_ptr(P, "P", true));
  if (tokens == 0) return AQUAKV_OK;
  const int d0 = which == AQUAKV_KEY ? d_in : d_in - D;
  const int d1 = which == AQUAKV_KEY ? 0 : D;
  HIP_TRY(aquakv::launch_predict(L->dtype, x0, d0, which == AQUAKV_KEY ? nullptr : x1, d1,
                                 which == AQUAKV_KEY ? L->w_k : L->w_v, which == AQUAKV_KEY ? L->b_k : L->b_v, P,
                                 tokens, D, static_cast<hipStream_t>(stream)));
  return AQUAKV_OK;
}

int aquakv_quantize(const aquakv_layer* L, int which, int64_t tokens, const void* X, const float* P, uint8_t* codes,
                    uint16_t* scales, void* Xhat, void* stream) {
  CHECK(check_layer(L));
  if (which != AQUAKV_KEY && which != AQUAKV_VALUE) return fail(AQUAKV_EINVAL, "which=%d", which);
  if (tokens < 0) return fail(AQUAKV_EINVAL, "tokens=%lld", (long long)tokens);
  CHECK(check_ptr(X, "X", true));
  CHECK(check_ptr(P, "P", false));
  CHECK(check_ptr(codes, "codes", true));
  CHECK(check_scales(L, scales, "scales", true));
  CHECK(check_ptr(Xhat, "Xhat", false));
  const aquakv::QuantizeIo io = {X, which == AQUAKV_KEY ? L->signs_k : L->signs_v, codes, scales, Xhat};
  const aquakv::Prediction pred = aquakv::Prediction::contiguous(P, L->kv_heads * L->head_dim);
  HIP_TRY(aquakv::launch_quantize(L->dtype, quantizer_id(L), &io, 1, P != nullptr ? &pred : nullptr, L->codebook, L->search_table, tokens, L->kv_heads,
                                  is_wide(L), static_cast<hipStream_t>(stream)));
  return AQUAKV_OK;
}

int aquakv_dequantize(const aquakv_layer* L, int which, int64_t tokens, const uint8_t* codes, const uint16_t* scales,
                      const float* P, void* Xhat, void* stream) {
  CHECK(check_layer(L));
  if (which != AQUAKV_KEY && which != AQUAKV_VALUE) return fail(AQUAKV_EINVAL, "which=%d", which);
  if (tokens < 0) return fail(AQUAKV_EINVAL, "tokens=%lld", (long long)tokens);
  CHECK(check_ptr(codes, "codes", true));
  CHECK(check_scales(L, scales, "scales", true));
  CHECK(check_ptr(P, "P", false));
  CHECK(check_ptr(Xhat, "Xhat", true));
  const aquakv::QuantizeIo io = coded(which == AQUAKV_KEY ? L->signs_k : L->signs_v, codes, scales, Xhat);
  HIP_TRY(aquakv::launch_dequantize(L->dtype, quantizer_id(L), &io, 1, P, L->codebook, tokens, L->kv_heads, is_wide(L),
                                    static_cast<hipStream_t>(stream)));
  return AQUAKV_OK;
}

int aquakv_encode_layer(const aquakv_layer* L, int64_t tokens, const void* K, const void* V, const void* Khat_prev,
                        const void* Vhat_prev, uint8_t* k_codes, uint16_t* k_scales, uint8_t* v_codes,
                        uint16_t* v_scales, void* Khat, void* Vhat, void* workspace, size_t workspace_bytes,
                        void* stream_) {
  CHECK(check_layer(L));
  if (tokens < 0) return fail(AQUAKV_EINVAL, "tokens=%lld", (long long)tokens);
  const bool has_k = L->d_in_k != 0, has_v = L->d_in_v != 0;
  CHECK(check_ptr(K, "K", true));
  CHECK(check_ptr(V, "V", true));
  CHECK(check_ptr(Khat_prev, "Khat_prev", has_k));
  CHECK(check_ptr(Vhat_prev, "Vhat_prev", has_v));
  CHECK(check_ptr(k_codes, "k_codes", true));
  CHECK(check_scales(L, k_scales, "k_scales", true));
  CHECK(check_ptr(v_codes, "v_codes", true));
  CHECK(check_scales(L, v_scales, "v_scales", true));
  CHECK(check_ptr(Khat, "Khat", false));
  CHECK(check_ptr(Vhat, "Vhat", false));
  if (tokens == 0) return AQUAKV_OK;
  const Plan pl = make_plan(L, tokens);
  CHECK(check_ptr(workspace, "workspace", true));
  if (workspace_bytes < pl.p_bytes + pl.khat_bytes)
    return fail(AQUAKV_EWORKSPACE, "workspace %zu B < required %zu B", workspace_bytes, pl.p_bytes + pl.khat_bytes);

  const size_t row = (size_t)pl.D * pl.eb;
  const bool khat_in_workspace = Khat == nullptr && has_v;
  size_t usable;
  bool at_once;
  {
    const size_t t = (size_t)tokens, crow = pl.code_row, srow = scale_row_bytes(L);
    const Range outs[] = {{Khat, t * row, "Khat"}, {Vhat, t * row, "Vhat"}, {k_codes, t * crow, "k_codes"},
                          {v_codes, t * crow, "v_codes"}, {k_scales, t * srow, "k_scales"}, {v_scales, t * srow, "v_scales"},
                          {workspace, pl.p_bytes + pl.khat_bytes, "workspace"}};
    const Range ins[] = {{K, t * row, "K"}, {V, t * row, "V"}, {Khat_prev, t * L->d_in_k * pl.eb, "Khat_prev"},
                         {Vhat_prev, has_v ? t * (L->d_in_v - pl.D) * pl.eb : 0, "Vhat_prev"}};
    const void* const inplace[] = {K, V, nullptr, nullptr, nullptr, nullptr, nullptr};
    CHECK(check_no_alias(outs, 7, ins, 4, inplace));
    usable = usable_workspace(L, pl, tokens, workspace, pl.p_bytes + (khat_in_workspace ? pl.khat_bytes : 0), pl.p_bytes + pl.khat_bytes,
                              workspace_bytes, outs, 6, ins, 4);
    // (half of the sums goes where a temporary Khat would lie)
    at_once = Khat != nullptr && !is_wide(L) && layer_at_once(L, pl, tokens, V, Vhat) &&
              clear_of(L, {workspace, t * row, ""}, outs, 6, ins, 4);
  }

  hipStream_t stream = static_cast<hipStream_t>(stream_);
  float* Pbuf = static_cast<float*>(workspace);
  // predictions at the front, the temporary Khat (if one is needed) at the back
  const size_t room = khat_in_workspace ? (usable - pl.khat_bytes) & ~(size_t)15 : usable;
  void* khat_tmp = static_cast<unsigned char*>(workspace) + room;

  if (at_once) {
    const aquakv::FusedTensor k = {Khat_prev, nullptr, L->d_in_k, 0, L->w_k, L->b_k, L->signs_k, K, k_codes, k_scales, Khat};
    const aquakv::FusedTensor v = {Vhat_prev, Khat, L->d_in_v - pl.D, pl.D, L->w_v, L->b_v, L->signs_v, V, v_codes, v_scales, Vhat};
    HIP_TRY(aquakv::launch_fused_layer(true, quantizer_id(L), L->codebook, L->search_table, k, v, workspace, tokens, pl.D, false, stream));
    return AQUAKV_OK;
  }
  for (int64_t r0 = 0; r0 < tokens; r0 += pl.chunk) {
    const int64_t n = tokens - r0 < pl.chunk ? tokens - r0 : pl.chunk;
    void* khat_dst = Khat != nullptr ? at(Khat, r0, row) : (has_v ? khat_tmp : nullptr);
    if (!has_k && !has_v) {                                 // nothing passes from the keys to the values: one launch
      const size_t srow = scale_row_bytes(L);
      const aquakv::QuantizeIo io[2] = {
          {at(K, r0, row), L->signs_k, static_cast<uint8_t*>(at(k_codes, r0, pl.code_row)),
           static_cast<uint16_t*>(at(k_scales, r0, srow)), khat_dst},
          {at(V, r0, row), L->signs_v, static_cast<uint8_t*>(at(v_codes, r0, pl.code_row)),
           static_cast<uint16_t*>(at(v_scales, r0, srow)), at(Vhat, r0, row)}};
      HIP_TRY(aquakv::launch_quantize(L->dtype, quantizer_id(L), io, 2, nullptr, L->codebook, L->search_table, n, L->kv_heads,
                                      is_wide(L), stream));
      continue;
    }
    CHECK(encode_keys_chunk(L, pl, r0, n, K, Khat_prev, k_codes, k_scales, khat_dst, Pbuf, room, stream));
    CHECK(encode_values_chunk(L, pl, r0, n, V, Vhat_prev, khat_dst, v_codes, v_scales, Vhat, Pbuf, room, stream));
  }
  return AQUAKV_OK;
}

int aquakv_decode_layer(const aquakv_layer* L, int64_t tokens, const uint8_t* k_codes, const uint16_t* k_scales,
                        const uint8_t* v_codes, const uint16_t* v_scales, const void* Khat_prev, const void* Vhat_prev,
                        void* Khat, void* Vhat, void* workspace, size_t workspace_bytes, void* stream_) {
  CHECK(check_layer(L));
  if (tokens < 0) return fail(AQUAKV_EINVAL, "tokens=%lld", (long long)tokens);
  const bool want_v = Vhat != nullptr;
  const bool has_k = L->d_in_k != 0, has_v = L->d_in_v != 0 && want_v;
  CHECK(check_ptr(k_codes, "k_codes", true));
  CHECK(check_scales(L, k_scales, "k_scales", true));
  CHECK(check_ptr(v_codes, "v_codes", want_v));
  CHECK(check_scales(L, v_scales, "v_scales", want_v));
  CHECK(check_ptr(Khat_prev, "Khat_prev", has_k));
  CHECK(check_ptr(Vhat_prev, "Vhat_prev", has_v));
  CHECK(check_ptr(Khat, "Khat", true));
  CHECK(check_ptr(Vhat, "Vhat", false));
  if (tokens == 0) return AQUAKV_OK;
  const Plan pl = make_plan(L, tokens);
  CHECK(check_ptr(workspace, "workspace", true));
  if (workspace_bytes < pl.p_bytes + pl.khat_bytes)
    return fail(AQUAKV_EWORKSPACE, "workspace %zu B < required %zu B", workspace_bytes, pl.p_bytes + pl.khat_bytes);

  bool at_once;
  {
    const size_t t = (size_t)tokens, row = (size_t)pl.D * pl.eb, crow = pl.code_row, srow = scale_row_bytes(L);
    const Range outs[] = {{Khat, t * row, "Khat"}, {Vhat, t * row, "Vhat"}, {workspace, pl.p_bytes, "workspace"}};
    const Range ins[] = {{Khat_prev, t * L->d_in_k * pl.eb, "Khat_prev"},
                         {Vhat_prev, has_v ? t * (L->d_in_v - pl.D) * pl.eb : 0, "Vhat_prev"},
                         {k_codes, t * crow, "k_codes"}, {v_codes, want_v ? t * crow : 0, "v_codes"},
                         {k_scales, t * srow, "k_scales"}, {v_scales, want_v ? t * srow : 0, "v_scales"}};
    CHECK(check_no_alias(outs, 3, ins, 6));
    at_once = layer_at_once(L, pl, tokens, nullptr, Vhat) && clear_of(L, {workspace, t * row, ""}, outs, 2, ins, 6);
  }
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  float* Pbuf = static_cast<float*>(workspace);
  if (at_once) {
    const aquakv::FusedTensor k = {Khat_prev, nullptr, L->d_in_k, 0, L->w_k, L->b_k, L->signs_k, nullptr,
                                   const_cast<uint8_t*>(k_codes), const_cast<uint16_t*>(k_scales), Khat};
    const aquakv::FusedTensor v = {Vhat_prev, Khat, L->d_in_v - pl.D, pl.D, L->w_v, L->b_v, L->signs_v, nullptr,
                                   const_cast<uint8_t*>(v_codes), const_cast<uint16_t*>(v_scales), Vhat};
    HIP_TRY(aquakv::launch_fused_layer(false, quantizer_id(L), L->codebook, nullptr, k, v, workspace, tokens, pl.D, is_wide(L), stream));
    return AQUAKV_OK;
  }

  for (int64_t r0 = 0; r0 < tokens; r0 += pl.chunk) {
    const int64_t n = tokens - r0 < pl.chunk ? tokens - r0 : pl.chunk;
    if (!has_k && want_v && !has_v) {                       // no predictors: keys and values in one launch
      const size_t row = (size_t)pl.D * pl.eb, srow = scale_row_bytes(L);
      const aquakv::QuantizeIo io[2] = {
          coded(L->signs_k, at(k_codes, r0, pl.code_row), at(k_scales, r0, srow), at(Khat, r0, row)),
          coded(L->signs_v, at(v_codes, r0, pl.code_row), at(v_scales, r0, srow), at(Vhat, r0, row))};
      HIP_TRY(aquakv::launch_dequantize(L->dtype, quantizer_id(L), io, 2, nullptr, L->codebook, n, L->kv_heads, is_wide(L), stream));
      continue;
    }
    CHECK(decode_keys_chunk(L, pl, r0, n, k_codes, k_scales, Khat_prev, Khat, Pbuf, stream));
    if (want_v) CHECK(decode_values_chunk(L, pl, r0, n, v_codes, v_scales, Vhat_prev, Khat, Vhat, Pbuf, stream));
  }
  return AQUAKV_OK;
}

// ---- a stack of layers ------------------------------------------------------------------------------------------
namespace {
// What aquakv_encode_layers checks of its arguments
int check_encode_layers(const aquakv_encode_entry* layers, int32_t n_layers, int64_t tokens, void* const* hat, const void* workspace,
                        size_t workspace_bytes) {
  if (layers == nullptr || hat == nullptr) return fail(AQUAKV_ENULL, "layers / hat is NULL");
  if (n_layers < 1) return fail(AQUAKV_EINVAL, "n_layers=%d", n_layers);
  if (tokens < 0) return fail(AQUAKV_EINVAL, "tokens=%lld", (long long)tokens);
  const aquakv_layer* first = nullptr;
  for (int32_t l = 0; l < n_layers; ++l) {
    const aquakv_encode_entry& c = layers[l];
    const aquakv_layer* const L = c.layer;
    CHECK(check_ptr(c.K, "K", true));
    CHECK(check_ptr(c.V, "V", true));
    if (L == nullptr) continue;
    CHECK(check_layer(L));
    if (first == nullptr) first = L;
    const int D = L->kv_heads * L->head_dim;
    if (L->kv_heads != first->kv_heads || L->dtype != first->dtype)
      return fail(AQUAKV_EINVAL, "layer %d: kv_heads=%d dtype=%d differ from those before", l, L->kv_heads, L->dtype);
    if ((L->d_in_k != 0 && L->d_in_k != D) || (L->d_in_v != 0 && L->d_in_v != 2 * D))
      return fail(AQUAKV_EINVAL, "layer %d: predictors of %d and %d inputs, layers of %d heads need %d and %d", l, L->d_in_k, L->d_in_v,
                  L->kv_heads, D, 2 * D);
    if (l == 0 && (L->d_in_k != 0 || L->d_in_v != 0)) return fail(AQUAKV_ENULL, "layer 0 has predictors, but no layer comes before it");
    CHECK(check_ptr(c.k_codes, "k_codes", true));
    CHECK(check_scales(L, c.k_scales, "k_scales", true));
    CHECK(check_ptr(c.v_codes, "v_codes", true));
    CHECK(check_scales(L, c.v_scales, "v_scales", true));
  }
  if (first == nullptr || tokens == 0) return AQUAKV_OK;
  for (int i = 0; i < 4; ++i) CHECK(check_ptr(hat[i], "hat", true));
  CHECK(check_ptr(workspace, "workspace", true));
  const size_t t = (size_t)tokens, row = (size_t)first->kv_heads * first->head_dim * elem_bytes(first->dtype);
  for (int32_t l = 0; l < n_layers; ++l) {
    if (layers[l].layer == nullptr) continue;
    const Plan pl = make_plan(layers[l].layer, tokens);
    if (workspace_bytes < pl.p_bytes + pl.khat_bytes)
      return fail(AQUAKV_EWORKSPACE, "workspace %zu B < required %zu B", workspace_bytes, pl.p_bytes + pl.khat_bytes);
  }
  const auto add = [](CacheRange* r, int64_t& n, const void* p, size_t bytes, const char* name, int32_t layer, bool written) {
    const uintptr_t begin = reinterpret_cast<uintptr_t>(p);
    if (p != nullptr && bytes != 0) r[n++] = {begin, begin + bytes, name, layer, written};
  };
  const auto add_codes = [&](CacheRange* r, int64_t& n, int32_t l) {
    const aquakv_encode_entry& c = layers[l];
    const size_t crow = make_plan(c.layer, 1).code_row, srow = scale_row_bytes(c.layer);
    add(r, n, c.k_codes, t * crow, "k_codes", l, true);
    add(r, n, c.k_scales, t * srow, "k_scales", l, true);
    add(r, n, c.v_codes, t * crow, "v_codes", l, true);
    add(r, n, c.v_scales, t * srow, "v_scales", l, true);
  };
  const auto add_common = [&](CacheRange* r, int64_t& n) {
    for (int i = 0; i < 4; ++i) add(r, n, hat[i], t * row, "hat", i >> 1, true);
    add(r, n, workspace, workspace_bytes, "workspace", 0, true);
  };
  for (int32_t l = 0; l < n_layers; ++l) {                   // a layer and the next one, with everything the call writes for all
    CacheRange r[4 + 1 + 2 * 6];
    int64_t n = 0;
    add_common(r, n);
    for (int32_t m = l; m < n_layers && m < l + 2; ++m) {
      add(r, n, layers[m].K, t * row, "K", m, false);
      add(r, n, layers[m].V, t * row, "V", m, false);
      if (layers[m].layer != nullptr) add_codes(r, n, m);
    }
    CHECK(check_disjoint(r, n));
  }
  // the parameters of all layers against all that is written; what a layer shares with the one before is there already
  const std::unique_ptr<CacheRange[]> ranges(new (std::nothrow) CacheRange[4 + 1 + (size_t)n_layers * (4 + 8)]);
  if (ranges == nullptr) return fail(AQUAKV_EINVAL, "no host memory to check %d layers", n_layers);
  int64_t n = 0;
  add_common(ranges.get(), n);
  Params before = {};
  for (int32_t l = 0; l < n_layers; ++l) {
    if (layers[l].layer == nullptr) continue;
    add_codes(ranges.get(), n, l);
    const Params params = params_of(layers[l].layer);
    for (int i = 0; i < 8; ++i)
      if (params.r[i].p != before.r[i].p || params.r[i].n != before.r[i].n)
        add(ranges.get(), n, params.r[i].p, params.r[i].n, params.r[i].name, l, false);
    before = params;
  }
  return check_disjoint(ranges.get(), n, true);
}
}  // namespace

int aquakv_encode_layers(const aquakv_encode_entry* layers, int32_t n_layers, int64_t tokens, void* const* hat, void* workspace,
                         size_t workspace_bytes, void* stream_) {
  CHECK(check_encode_layers(layers, n_layers, tokens, hat, workspace, workspace_bytes));
  if (tokens == 0) return AQUAKV_OK;
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  float* const ws = static_cast<float*>(workspace);
  // values of layer l and keys of layer l + 1 at once: bf16, one quantizer, few rows
  const auto with_next = [&](int32_t l) {
    const aquakv_layer *a = layers[l].layer, *b = l + 1 < n_layers ? layers[l + 1].layer : nullptr;
    if (a == nullptr || b == nullptr || a->dtype != AQUAKV_BF16 || a->d_in_v == 0 || b->d_in_k == 0 ||
        quantizer_id(a) != quantizer_id(b) || is_wide(a) != is_wide(b))
      return false;
    const int D = a->kv_heads * 128;
    if (!is_wide(a)) return aquakv::fused_encode_pair_pays(tokens, D);
    return tokens <= aquakv::tile_predict_pair_rows(D) && workspace_bytes >= 2 * (size_t)tokens * D * elem_bytes(a->dtype);
  };
  const auto keys_hat = [&](int32_t l) { return hat[2 * (l & 1)]; };
  const auto values_hat = [&](int32_t l) { return hat[2 * (l & 1) + 1]; };
  const void *Kp = nullptr, *Vp = nullptr;                   // of the layer before
  const auto key_tensor = [&](int32_t l, const void* prev) {
    const aquakv_encode_entry& c = layers[l];
    return aquakv::FusedTensor{prev, nullptr, c.layer->d_in_k, 0, c.layer->w_k, c.layer->b_k, c.layer->signs_k, c.K, c.k_codes, c.k_scales,
                               keys_hat(l)};
  };
  bool have_keys = false;                                    // of this layer, encoded with the values of the one before
  for (int32_t l = 0; l < n_layers; ++l) {
    const aquakv_encode_entry& c = layers[l];
    const aquakv_layer* const L = c.layer;
    if (L == nullptr) {
      Kp = c.K; Vp = c.V;
      continue;
    }
    const int D = L->kv_heads * L->head_dim;
    const Plan pl = make_plan(L, tokens);
    void *const K = keys_hat(l), *const V = values_hat(l);
    const bool pair = with_next(l);
    if (!have_keys && !pair) {
      CHECK(aquakv_encode_layer(L, tokens, c.K, c.V, Kp, Vp, c.k_codes, c.k_scales, c.v_codes, c.v_scales, K, V, workspace,
                                workspace_bytes, stream));
    } else {
      const size_t row = (size_t)D * pl.eb;
      for (int64_t r0 = 0; r0 < tokens && !have_keys; r0 += pl.chunk)
        CHECK(encode_keys_chunk(L, pl, r0, tokens - r0 < pl.chunk ? tokens - r0 : pl.chunk, c.K, Kp, c.k_codes, c.k_scales,
                                at(K, r0, row), ws, workspace_bytes, stream));
      if (!pair) {
        for (int64_t r0 = 0; r0 < tokens; r0 += pl.chunk)
          CHECK(encode_values_chunk(L, pl, r0, tokens - r0 < pl.chunk ? tokens - r0 : pl.chunk, c.V, Vp, at(K, r0, row), c.v_codes,
                                    c.v_scales, V, ws, workspace_bytes, stream));
      } else {
        const aquakv_layer* const N = layers[l + 1].layer;
        const aquakv::FusedTensor t[2] = {
            {Vp, K, D, D, L->w_v, L->b_v, L->signs_v, c.V, c.v_codes, c.v_scales, V}, key_tensor(l + 1, K)};
        const float* const codebooks[2] = {L->codebook, N->codebook};
        const void* const tables[2] = {L->search_table, N->search_table};
        if (!is_wide(L)) {
          HIP_TRY(aquakv::launch_fused_encode_pair(quantizer_id(L), t, codebooks, tables, tokens, D, stream));
        } else {
          // predictions in fp32, the upper heads' in the workspace and the others' in the rows that the quantizer will write
          aquakv::Prediction P[2];
          aquakv::QuantizeIo io[2];
          for (int i = 0; i < 2; ++i) {
            P[i] = {static_cast<float*>(t[i].Xhat), ws + i * tokens * (D / 2), D / 2, D / 2};
            io[i] = {t[i].X, t[i].signs, t[i].codes, t[i].scales, t[i].Xhat};
          }
          HIP_TRY(aquakv::launch_tile_predict_pair(t, P, tokens, D, stream));
          const bool one = is_rtn(L) || (codebooks[0] == codebooks[1] && tables[0] == tables[1]);
          for (int i = 0; i < (one ? 1 : 2); ++i)
            HIP_TRY(aquakv::launch_quantize(L->dtype, quantizer_id(L), io + i, one ? 2 : 1, P + i, codebooks[i], tables[i], tokens,
                                            L->kv_heads, true, stream));
        }
      }
    }
    have_keys = pair;
    Kp = K; Vp = V;
  }
  return AQUAKV_OK;
}

// ---- the two halves of Alg. "encode" / "decode" as calls of their own -------------------------------------------
// The key chain of a layer stack depends on keys only, the value chain on the previous values and this layer's keys,
// so a caller can run them on two streams (events between them) and overlap the kernels of neighbouring layers.
int aquakv_encode_keys(const aquakv_layer* L, int64_t tokens, const void* K, const void* Khat_prev, uint8_t* k_codes,
                       uint16_t* k_scales, void* Khat, void* workspace, size_t workspace_bytes, void* stream_) {
  CHECK(check_layer(L));
  if (tokens < 0) return fail(AQUAKV_EINVAL, "tokens=%lld", (long long)tokens);
  CHECK(check_ptr(K, "K", true));
  CHECK(check_ptr(Khat_prev, "Khat_prev", L->d_in_k != 0));
  CHECK(check_ptr(k_codes, "k_codes", true));
  CHECK(check_scales(L, k_scales, "k_scales", true));
  CHECK(check_ptr(Khat, "Khat", false));
  if (tokens == 0) return AQUAKV_OK;
  const Plan pl = make_plan(L, tokens);
  if (pl.p_bytes != 0) {
    CHECK(check_ptr(workspace, "workspace", true));
    if (workspace_bytes < pl.p_bytes) return fail(AQUAKV_EWORKSPACE, "workspace %zu B < required %zu B", workspace_bytes, pl.p_bytes);
  }
  const size_t row = (size_t)pl.D * pl.eb;
  size_t room;
  {
    const size_t t = (size_t)tokens;
    const Range outs[] = {{Khat, t * row, "Khat"}, {k_codes, t * pl.code_row, "k_codes"},
                          {k_scales, t * scale_row_bytes(L), "k_scales"}, {workspace, pl.p_bytes, "workspace"}};
    const Range ins[] = {{K, t * row, "K"}, {Khat_prev, t * L->d_in_k * pl.eb, "Khat_prev"}};
    const void* const inplace[] = {K, nullptr, nullptr, nullptr};
    CHECK(check_no_alias(outs, 4, ins, 2, inplace));
    room = pl.p_bytes == 0 ? 0 : usable_workspace(L, pl, tokens, workspace, pl.p_bytes, pl.p_bytes, workspace_bytes, outs, 3, ins, 2);
  }
  for (int64_t r0 = 0; r0 < tokens; r0 += pl.chunk) {
    const int64_t n = tokens - r0 < pl.chunk ? tokens - r0 : pl.chunk;
    CHECK(encode_keys_chunk(L, pl, r0, n, K, Khat_prev, k_codes, k_scales, at(Khat, r0, row), static_cast<float*>(workspace),
                            room, static_cast<hipStream_t>(stream_)));
  }
  return AQUAKV_OK;
}

int aquakv_encode_values(const aquakv_layer* L, int64_t tokens, const void* V, const void* Vhat_prev, const void* Khat,
                         uint8_t* v_codes, uint16_t* v_scales, void* Vhat, void* workspace, size_t workspace_bytes,
                         void* stream_) {
  CHECK(check_layer(L));
  if (tokens < 0) return fail(AQUAKV_EINVAL, "tokens=%lld", (long long)tokens);
  const bool has_v = L->d_in_v != 0;
  CHECK(check_ptr(V, "V", true));
  CHECK(check_ptr(Vhat_prev, "Vhat_prev", has_v));
  CHECK(check_ptr(Khat, "Khat", has_v));
  CHECK(check_ptr(v_codes, "v_codes", true));
  CHECK(check_scales(L, v_scales, "v_scales", true));
  CHECK(check_ptr(Vhat, "Vhat", false));
  if (tokens == 0) return AQUAKV_OK;
  const Plan pl = make_plan(L, tokens);
  if (pl.p_bytes != 0) {
    CHECK(check_ptr(workspace, "workspace", true));
    if (workspace_bytes < pl.p_bytes) return fail(AQUAKV_EWORKSPACE, "workspace %zu B < required %zu B", workspace_bytes, pl.p_bytes);
  }
  const size_t row = (size_t)pl.D * pl.eb;
  size_t room;
  {
    const size_t t = (size_t)tokens;
    const Range outs[] = {{Vhat, t * row, "Vhat"}, {v_codes, t * pl.code_row, "v_codes"},
                          {v_scales, t * scale_row_bytes(L), "v_scales"}, {workspace, pl.p_bytes, "workspace"}};
    const Range ins[] = {{V, t * row, "V"}, {Vhat_prev, has_v ? t * (L->d_in_v - pl.D) * pl.eb : 0, "Vhat_prev"},
                         {Khat, has_v ? t * row : 0, "Khat"}};
    const void* const inplace[] = {V, nullptr, nullptr, nullptr};
    CHECK(check_no_alias(outs, 4, ins, 3, inplace));
    room = pl.p_bytes == 0 ? 0 : usable_workspace(L, pl, tokens, workspace, pl.p_bytes, pl.p_bytes, workspace_bytes, outs, 3, ins, 3);
  }
  for (int64_t r0 = 0; r0 < tokens; r0 += pl.chunk) {
    const int64_t n = tokens - r0 < pl.chunk ? tokens - r0 : pl.chunk;
    CHECK(encode_values_chunk(L, pl, r0, n, V, Vhat_prev, at(Khat, r0, row), v_codes, v_scales, Vhat,
                              static_cast<float*>(workspace), room, static_cast<hipStream_t>(stream_)));
  }
  return AQUAKV_OK;
}

int aquakv_decode_values(const aquakv_layer* L, int64_t tokens, const uint8_t* v_codes, const uint16_t* v_scales,
                         const void* Vhat_prev, const void* Khat, void* Vhat, void* workspace, size_t workspace_bytes,
                         void* stream_) {
  CHECK(check_layer(L));
  if (tokens < 0) return fail(AQUAKV_EINVAL, "tokens=%lld", (long long)tokens);
  const bool has_v = L->d_in_v != 0;
  CHECK(check_ptr(v_codes, "v_codes", true));
  CHECK(check_scales(L, v_scales, "v_scales", true));
  CHECK(check_ptr(Vhat_prev, "Vhat_prev", has_v));
  CHECK(check_ptr(Khat, "Khat", has_v));
  CHECK(check_ptr(Vhat, "Vhat", true));
  if (tokens == 0) return AQUAKV_OK;
  const Plan pl = make_plan(L, tokens);
  if (pl.p_bytes != 0) {
    CHECK(check_ptr(workspace, "workspace", true));
    if (workspace_bytes < pl.p_bytes) return fail(AQUAKV_EWORKSPACE, "workspace %zu B < required %zu B", workspace_bytes, pl.p_bytes);
  }
  {
    const size_t t = (size_t)tokens, row = (size_t)pl.D * pl.eb;
    const Range outs[] = {{Vhat, t * row, "Vhat"}, {workspace, pl.p_bytes, "workspace"}};
    const Range ins[] = {{Vhat_prev, has_v ? t * (L->d_in_v - pl.D) * pl.eb : 0, "Vhat_prev"}, {Khat, has_v ? t * row : 0, "Khat"},
                         {v_codes, t * pl.code_row, "v_codes"}, {v_scales, t * scale_row_bytes(L), "v_scales"}};
    CHECK(check_no_alias(outs, 2, ins, 4));
  }
  for (int64_t r0 = 0; r0 < tokens; r0 += pl.chunk) {
    const int64_t n = tokens - r0 < pl.chunk ? tokens - r0 : pl.chunk;
    CHECK(decode_values_chunk(L, pl, r0, n, v_codes, v_scales, Vhat_prev, Khat, Vhat, static_cast<float*>(workspace),
                              static_cast<hipStream_t>(stream_)));
  }
  return AQUAKV_OK;
}

// ---- value side of attention: soft-max rows, decode of the values with the weighted sum over tokens ------------
namespace {
size_t weighted_part_bytes(int32_t batch, int32_t seq_len, int32_t q_heads) {
  const size_t chunks = ((size_t)seq_len + aquakv::kWeightedChunk - 1) / aquakv::kWeightedChunk;
  const size_t bytes = (size_t)batch * chunks * q_heads * 128 * sizeof(float);
  return (bytes + 255) & ~(size_t)255;
}
size_t weighted_stat_bytes(int32_t batch, int32_t seq_len, int32_t q_heads) {
  const size_t chunks = ((size_t)seq_len + aquakv::kWeightedChunk - 1) / aquakv::kWeightedChunk;
  const size_t bytes = (size_t)batch * chunks * q_heads * 2 * sizeof(float);
  return (bytes + 255) & ~(size_t)255;
}
bool weighted_fused(const aquakv_layer* L, const Plan& pl, int32_t seq_len) {
  return L->d_in_v != 0 && pl.fused_dec && seq_len % aquakv::kWeightedChunk == 0;
}
}  // namespace

int aquakv_softmax(int64_t rows, int64_t n, const float* scores, float* probs, void* stream) {
  if (rows < 0 || n < 0 || rows > 0x7fffffffLL) return fail(AQUAKV_EINVAL, "rows=%lld n=%lld", (long long)rows, (long long)n);
  CHECK(check_ptr(scores, "scores", true));
  CHECK(check_ptr(probs, "probs", true));
  HIP_TRY(aquakv::launch_softmax_rows(scores, probs, rows, n, static_cast<hipStream_t>(stream)));
  return AQUAKV_OK;
}

size_t aquakv_weighted_workspace_bytes(const aquakv_layer* L, int32_t batch, int32_t seq_len, int32_t q_heads) {
  if (check_layer(L) != AQUAKV_OK || batch < 1 || seq_len < 1 || q_heads < 1) return 0;
  const Plan pl = make_plan(L, (int64_t)batch * seq_len);
  return weighted_part_bytes(batch, seq_len, q_heads) + weighted_stat_bytes(batch, seq_len, q_heads) + pl.p_bytes;
}

namespace {
// shared body: softmax = false: `weights` are the weights; true: they are raw scores (soft-max taken per chunk and merged)
int decode_values_weighted(const aquakv_layer* L, int32_t batch, int32_t seq_len, int32_t q_heads, const uint8_t* v_codes,
                           const uint16_t* v_scales, const void* Vhat_prev, const void* Khat, const float* weights,
                           bool softmax, void* Vhat, float* out, float* row_stats, void* workspace, size_t workspace_bytes,
                           void* stream_) {
  CHECK(check_layer(L));
  if (batch < 0 || seq_len < 0) return fail(AQUAKV_EINVAL, "batch=%d seq_len=%d", batch, seq_len);
  if (q_heads < 1 || q_heads % L->kv_heads || q_heads / L->kv_heads > 8)
    return fail(AQUAKV_EINVAL, "q_heads=%d must be a multiple of kv_heads=%d, at most 8x", q_heads, L->kv_heads);
  const bool has_v = L->d_in_v != 0;
  CHECK(check_ptr(v_codes, "v_codes", true));
  CHECK(check_scales(L, v_scales, "v_scales", true));
  CHECK(check_ptr(Vhat_prev, "Vhat_prev", has_v));
  CHECK(check_ptr(Khat, "Khat", has_v));
  CHECK(check_ptr(weights, softmax ? "scores" : "weights", true));
  CHECK(check_ptr(Vhat, "Vhat", false));
  CHECK(check_ptr(out, "out", true));
  if (row_stats != nullptr && (reinterpret_cast<uintptr_t>(row_stats) & 3u))
    return fail(AQUAKV_EALIGN, "row_stats is not 4-byte aligned");
  const int64_t tokens = (int64_t)batch * seq_len;
  if (tokens == 0) return AQUAKV_OK;
  const Plan pl = make_plan(L, tokens);
  const bool fused = weighted_fused(L, pl, seq_len);
  if (!fused && Vhat == nullptr)
    return fail(AQUAKV_ENULL, "Vhat may be NULL only when the sums are taken inside the decode kernel (bf16, "
                              "a value predictor, seq_len a multiple of %d)",
                aquakv::kWeightedChunk);
  const size_t part_bytes = weighted_part_bytes(batch, seq_len, q_heads);
  const size_t stat_bytes = weighted_stat_bytes(batch, seq_len, q_heads);
  const size_t need = part_bytes + stat_bytes + (fused ? 0 : pl.p_bytes);
  CHECK(check_ptr(workspace, "workspace", true));
  if (workspace_bytes < need) return fail(AQUAKV_EWORKSPACE, "workspace %zu B < required %zu B", workspace_bytes, need);
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  unsigned char* wsb = static_cast<unsigned char*>(workspace);
  float* part = reinterpret_cast<float*>(wsb);
  float* pstats = softmax ? reinterpret_cast<float*>(wsb + part_bytes) : nullptr;
  float* Pbuf = reinterpret_cast<float*>(wsb + part_bytes + stat_bytes);
  if (fused) {
    const int D = pl.D;
    HIP_TRY(aquakv::launch_fused_weighted(quantizer_id(L), Vhat_prev, L->d_in_v - D, Khat, D, L->w_v, L->b_v, L->signs_v,
                                          L->codebook, v_codes, v_scales, Vhat, weights, part, pstats, seq_len, q_heads,
                                          tokens, D, is_wide(L), stream));
  } else {
    for (int64_t r0 = 0; r0 < tokens; r0 += pl.chunk) {
      const int64_t n = tokens - r0 < pl.chunk ? tokens - r0 : pl.chunk;
      CHECK(decode_values_chunk(L, pl, r0, n, v_codes, v_scales, Vhat_prev, Khat, Vhat, Pbuf, stream));
    }
    // sequences of one chunk (up to 256 tokens): the sums are the result and the launch that merges them is
    // saved: one layer of attention over 150 tokens 24.9 us against 27.2, 12 x 200 tokens 40.5 against 42.8
    const bool whole = seq_len <= aquakv::kWeightedChunk;
    const aquakv::WeightedForm form = !softmax ? aquakv::kWeightedGiven : whole ? aquakv::kWeightedWhole : aquakv::kWeightedSoftMax;
    HIP_TRY(aquakv::launch_weighted_values(L->dtype, Vhat, weights, form, whole ? out : part, whole ? (softmax ? row_stats : nullptr) : pstats,
                                           batch, seq_len, L->kv_heads, q_heads, stream));
    if (whole) return AQUAKV_OK;
  }
  HIP_TRY(aquakv::launch_combine_weighted(part, pstats, out, softmax ? row_stats : nullptr, batch, seq_len, q_heads, stream));
  return AQUAKV_OK;
}
}  // namespace

int aquakv_decode_values_weighted(const aquakv_layer* L, int32_t batch, int32_t seq_len, int32_t q_heads,
                                  const uint8_t* v_codes, const uint16_t* v_scales, const void* Vhat_prev,
                                  const void* Khat, const float* weights, void* Vhat, float* out, void* workspace,
                                  size_t workspace_bytes, void* stream) {
  return decode_values_weighted(L, batch, seq_len, q_heads, v_codes, v_scales, Vhat_prev, Khat, weights, false, Vhat, out,
                                nullptr, workspace, workspace_bytes, stream);
}

int aquakv_decode_values_attend(const aquakv_layer* L, int32_t batch, int32_t seq_len, int32_t q_heads,
                                const uint8_t* v_codes, const uint16_t* v_scales, const void* Vhat_prev, const void* Khat,
                                const float* scores, void* Vhat, float* out, float* row_stats, void* workspace,
                                size_t workspace_bytes, void* stream) {
  return decode_values_weighted(L, batch, seq_len, q_heads, v_codes, v_scales, Vhat_prev, Khat, scores, true, Vhat, out,
                                row_stats, workspace, workspace_bytes, stream);
}

int aquakv_attend_raw(int32_t dtype, int32_t batch, int32_t tokens, int32_t kv_heads, int32_t q_heads, const void* K,
                      const void* V, const void* q, const float* rope_cos, const float* rope_sin, float score_scale,
                      float* out, float* row_stats, int32_t accumulate, void* stream) {
  if (dtype != AQUAKV_BF16 && dtype != AQUAKV_FP32) return fail(AQUAKV_EINVAL, "dtype=%d", dtype);
  if (batch < 0 || tokens < 0) return fail(AQUAKV_EINVAL, "batch=%d tokens=%d", batch, tokens);
  if (tokens > aquakv::kAttendRawMaxTokens)
    return fail(AQUAKV_EUNSUPPORTED, "tokens=%d: at most %d uncompressed tokens per call", tokens, aquakv::kAttendRawMaxTokens);
  if (kv_heads < 1 || q_heads < 1 || q_heads % kv_heads)
    return fail(AQUAKV_EINVAL, "q_heads=%d must be a multiple of kv_heads=%d", q_heads, kv_heads);
  CHECK(check_ptr(K, "K", tokens != 0));
  CHECK(check_ptr(V, "V", tokens != 0));
  CHECK(check_ptr(q, "q", true));
  CHECK(check_ptr(out, "out", true));
  CHECK(check_ptr(row_stats, "row_stats", true));
  if ((rope_cos == nullptr) != (rope_sin == nullptr)) return fail(AQUAKV_ENULL, "rope_cos and rope_sin go together");
  CHECK(check_ptr(rope_cos, "rope_cos", false));
  CHECK(check_ptr(rope_sin, "rope_sin", false));
  if (batch == 0) return AQUAKV_OK;
  if (tokens == 0) {
    if (!accumulate) return fail(AQUAKV_EINVAL, "tokens=0 leaves nothing to write without a result to merge into");
    return AQUAKV_OK;
  }
  HIP_TRY(aquakv::launch_attend_raw(dtype, K, V, q, rope_cos, rope_sin, score_scale, out, row_stats, batch, tokens, kv_heads,
                                    q_heads, accumulate != 0, static_cast<hipStream_t>(stream)));
  return AQUAKV_OK;
}

// ---- calibration: ridge least-squares fit of one predictor (Alg. "Calibration") --------------------------------
size_t aquakv_fit_workspace_bytes(int32_t d_in, int32_t d_out) {
  if (d_in < 64 || d_in > 8192 || d_in % 64 || d_out < 64 || d_out > 8192 || d_out % 64) return 0;
  return aquakv::fit_workspace_bytes(d_in, d_out);
}

int aquakv_fit_predictor(int32_t dtype, int64_t tokens, const void* x0, int32_t d0, const void* x1, int32_t d1,
                         const void* Y, int32_t d_out, double rate, void* W, double* W64, float* bias, void* workspace,
                         size_t workspace_bytes, void* stream) {
  if (dtype != AQUAKV_BF16 && dtype != AQUAKV_FP32) return fail(AQUAKV_EINVAL, "dtype=%d", dtype);
  if (tokens < 1) return fail(AQUAKV_EINVAL, "tokens=%lld: at least one row is needed", (long long)tokens);
  if (d0 < 64 || d0 % 64 || d1 < 0 || d1 % 64) return fail(AQUAKV_EINVAL, "d0=%d d1=%d must be multiples of 64, d0 >= 64", d0, d1);
  if (d_out < 64 || d_out % 64) return fail(AQUAKV_EINVAL, "d_out=%d must be a positive multiple of 64", d_out);
  if ((int64_t)d0 + d1 > 8192 || d_out > 8192) return fail(AQUAKV_EUNSUPPORTED, "at most 8192 inputs and outputs");
  if (!(rate >= 0.0) || rate > 1e6) return fail(AQUAKV_EINVAL, "rate=%g", rate);
  CHECK(check_ptr(x0, "x0", true));
  CHECK(check_ptr(x1, "x1", d1 != 0));
  CHECK(check_ptr(Y, "Y", true));
  CHECK(check_ptr(W, "W", true));
  CHECK(check_ptr(W64, "W64", false));
  CHECK(check_ptr(bias, "bias", false));
  CHECK(check_ptr(workspace, "workspace", true));
  const size_t need = aquakv::fit_workspace_bytes(d0 + d1, d_out);
  if (workspace_bytes < need) return fail(AQUAKV_EWORKSPACE, "workspace %zu B < required %zu B", workspace_bytes, need);
  HIP_TRY(aquakv::launch_fit_predictor(dtype, tokens, x0, d0, d1 != 0 ? x1 : nullptr, d1, Y, d_out, rate, W, W64, bias, workspace,
                                       static_cast<hipStream_t>(stream)));
  return AQUAKV_OK;
}

int aquakv_copy_ranges(const aquakv_copy_range* ranges, int32_t n, void* stream) {
  if (n < 0) return fail(AQUAKV_EINVAL, "n=%d", n);
  if (n == 0) return AQUAKV_OK;
  if (ranges == nullptr) return fail(AQUAKV_ENULL, "ranges is NULL");
  static_assert(sizeof(aquakv_copy_range) == sizeof(aquakv::CopyRange), "same layout");
  for (int32_t i = 0; i < n; ++i)
    if (ranges[i].bytes != 0 && (ranges[i].dst == nullptr || ranges[i].src == nullptr))
      return fail(AQUAKV_ENULL, "range %d has a NULL pointer", i);
  HIP_TRY(aquakv::launch_copy_ranges(reinterpret_cast<const aquakv::CopyRange*>(ranges), n, static_cast<hipStream_t>(stream)));
  return AQUAKV_OK;
}

size_t aquakv_scores_workspace_bytes(const aquakv_layer* L, int32_t batch, int32_t q_heads) {
  if (check_layer(L) != AQUAKV_OK || batch < 1 || q_heads < 1) return 0;
  if (L->dtype != AQUAKV_BF16 || is_wide(L) || !aquakv::folded_scores_supported(L->kv_heads, L->d_in_k, q_heads)) return 0;
  return aquakv::folded_scores_workspace_bytes(batch, q_heads);
}

}  // extern "C"

namespace {
// The folded form keeps per-call operands (the folded queries) in device memory.  Callers that cannot allocate
// take them from this array instead of a workspace of their own: aquakv_decode_attn_scores_folded_static.
// Host code never uses the array's name as an address: the device address is asked for once per device
// (hipGetSymbolAddress, with that device current) and kept.
constexpr int kStaticFoldBatches = 64;                                    // batch x passes of one call
constexpr size_t kStaticFoldBytes = (size_t)kStaticFoldBatches * aquakv::kFoldedBytesPerBatch;   // about 9 MiB
__device__ __align__(256) unsigned char scratch[kStaticFoldBytes];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// device address of `scratch` on the current device (looked up on the first call per device)
int static_scratch(void** out) {
  int dev = -1;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(AQUAKV_EUNSUPPORTED, "device ordinal %d: at most %d devices", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* ptr = nullptr;
    HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (ptr == nullptr) return fail(AQUAKV_EHIP, "hipGetSymbolAddress returned a null address");
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return AQUAKV_OK;
}

enum ScoresForm { kFormDefinition = 0, kFormFolded = 1 };

// shared body of the scoring entry points; rope_cos / rope_sin both NULL: no rotary embedding
int decode_attn_scores(const aquakv_layer* L, int32_t batch, int32_t seq_len, int32_t q_heads, const uint8_t* k_codes,
                       const uint16_t* k_scales, const void* Khat_prev, const void* q, const float* rope_cos,
                       const float* rope_sin, float score_scale, float* scores, void* Khat_out, void* workspace,
                       size_t workspace_bytes, void* stream_, int form) {
  CHECK(check_layer(L));
  if (batch < 0 || seq_len < 0) return fail(AQUAKV_EINVAL, "batch=%d seq_len=%d", batch, seq_len);
  if (q_heads < 1 || q_heads % L->kv_heads || q_heads / L->kv_heads > 8)
    return fail(AQUAKV_EINVAL, "q_heads=%d must be a multiple of kv_heads=%d, at most 8x", q_heads, L->kv_heads);
  const bool has_k = L->d_in_k != 0;
  CHECK(check_ptr(k_codes, "k_codes", true));
  CHECK(check_scales(L, k_scales, "k_scales", true));
  CHECK(check_ptr(Khat_prev, "Khat_prev", has_k));
  CHECK(check_ptr(q, "q", true));
  CHECK(check_ptr(scores, "scores", true));
  CHECK(check_ptr(Khat_out, "Khat_out", false));
  const int64_t tokens = (int64_t)batch * seq_len;
  const Plan pl = make_plan(L, tokens > 0 ? tokens : 1);
  if (form == kFormFolded) {
    if (!(has_k && pl.fused && !is_wide(L) && aquakv::folded_scores_supported(L->kv_heads, L->d_in_k, q_heads)))
      return fail(AQUAKV_EUNSUPPORTED, "the folded form is built for bf16 layers with 8 kv heads, a key predictor with 1024 "
                                       "inputs, rotation groups of one head and at most 64 query heads");
    if (tokens == 0) return AQUAKV_OK;
    // predictor folded into the query: Khat_prev and the codes are read once, nothing is recomputed
    CHECK(check_ptr(workspace, "workspace", true));
    const size_t need = aquakv::folded_scores_workspace_bytes(batch, q_heads);
    if (workspace_bytes < need) return fail(AQUAKV_EWORKSPACE, "workspace %zu B < required %zu B", workspace_bytes, need);
    // the round-to-nearest backbone has neither rotation nor grid: whatever the layer holds there is not passed on
    HIP_TRY(aquakv::launch_folded_scores(quantizer_id(L), Khat_prev, L->w_k, L->b_k, is_rtn(L) ? nullptr : L->signs_k,
                                         is_rtn(L) ? nullptr : L->codebook, k_codes, k_scales, q, score_scale, scores,
                                         workspace, batch, seq_len, q_heads, static_cast<hipStream_t>(stream_)));
    return AQUAKV_OK;
  }
  if (tokens == 0) return AQUAKV_OK;
  if (has_k && pl.fused_dec) {
    // one fused launch over all rows: prediction, inverse quantizer and dot products
    HIP_TRY(aquakv::launch_fused_scores(quantizer_id(L), Khat_prev, L->d_in_k, L->w_k, L->b_k, L->signs_k, L->codebook,
                                        k_codes, k_scales, q, score_scale, scores, Khat_out, seq_len, q_heads, tokens,
                                        pl.D, rope_cos, rope_sin, is_wide(L), static_cast<hipStream_t>(stream_)));
    return AQUAKV_OK;
  }
  if (has_k) {
    CHECK(check_ptr(workspace, "workspace", true));
    if (workspace_bytes < pl.p_bytes)
      return fail(AQUAKV_EWORKSPACE, "workspace %zu B < required %zu B", workspace_bytes, pl.p_bytes);
  }
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  float* Pbuf = static_cast<float*>(workspace);
  const size_t row = (size_t)pl.D * pl.eb;
  const size_t srow = scale_row_bytes(L);
  for (int64_t r0 = 0; r0 < tokens; r0 += pl.chunk) {
    const int64_t n = tokens - r0 < pl.chunk ? tokens - r0 : pl.chunk;
    if (has_k)
      HIP_TRY(aquakv::launch_predict(L->dtype, at(Khat_prev, r0, (size_t)L->d_in_k * pl.eb), L->d_in_k, nullptr, 0,
                                     L->w_k, L->b_k, Pbuf, n, pl.D, stream));
    HIP_TRY(aquakv::launch_attn_scores(L->dtype, quantizer_id(L), static_cast<const uint8_t*>(at(k_codes, r0, pl.code_row)),
                                       static_cast<const uint16_t*>(at(k_scales, r0, srow)), has_k ? Pbuf : nullptr,
                                       L->signs_k, L->codebook, q, score_scale, scores, at(Khat_out, r0, row), r0, n,
                                       seq_len, L->kv_heads, q_heads, rope_cos, rope_sin, is_wide(L), stream));
  }
  return AQUAKV_OK;
}
}  // namespace

extern "C" {

int aquakv_decode_attn_scores(const aquakv_layer* L, int32_t batch, int32_t seq_len, int32_t q_heads,
                              const uint8_t* k_codes, const uint16_t* k_scales, const void* Khat_prev, const void* q,
                              float score_scale, float* scores, void* Khat_out, void* workspace,
                              size_t workspace_bytes, void* stream_) {
  return decode_attn_scores(L, batch, seq_len, q_heads, k_codes, k_scales, Khat_prev, q, nullptr, nullptr, score_scale,
                            scores, Khat_out, workspace, workspace_bytes, stream_, kFormDefinition);
}

int aquakv_decode_attn_scores_folded(const aquakv_layer* L, int32_t batch, int32_t seq_len, int32_t q_heads,
                                     const uint8_t* k_codes, const uint16_t* k_scales, const void* Khat_prev,
                                     const void* q, float score_scale, float* scores, void* workspace,
                                     size_t workspace_bytes, void* stream_) {
  return decode_attn_scores(L, batch, seq_len, q_heads, k_codes, k_scales, Khat_prev, q, nullptr, nullptr, score_scale,
                            scores, nullptr, workspace, workspace_bytes, stream_, kFormFolded);
}

int aquakv_decode_attn_scores_folded_static(const aquakv_layer* L, int32_t batch, int32_t seq_len, int32_t q_heads,
                                            const uint8_t* k_codes, const uint16_t* k_scales, const void* Khat_prev,
                                            const void* q, float score_scale, float* scores, void* stream_) {
  CHECK(check_layer(L));
  if (batch < 0 || q_heads < 1) return fail(AQUAKV_EINVAL, "batch=%d q_heads=%d", batch, q_heads);
  const size_t need = aquakv::folded_scores_workspace_bytes(batch, q_heads);
  if (need > kStaticFoldBytes)
    return fail(AQUAKV_EUNSUPPORTED, "batch=%d with %d query heads needs %zu B of folded queries; the built-in buffer holds "
                                     "%zu B (batch x passes <= %d, one pass per 32 query heads): use "
                                     "aquakv_decode_attn_scores_folded with a workspace",
                batch, q_heads, need, kStaticFoldBytes, kStaticFoldBatches);
  void* ptr = nullptr;
  CHECK(static_scratch(&ptr));
  return decode_attn_scores(L, batch, seq_len, q_heads, k_codes, k_scales, Khat_prev, q, nullptr, nullptr, score_scale,
                            scores, nullptr, ptr, kStaticFoldBytes, stream_, kFormFolded);
}

int aquakv_decode_attn_scores_rope(const aquakv_layer* L, int32_t batch, int32_t seq_len, int32_t q_heads,
                                   const uint8_t* k_codes, const uint16_t* k_scales, const void* Khat_prev,
                                   const void* q, const float* rope_cos, const float* rope_sin, float score_scale,
                                   float* scores, void* Khat_out, void* workspace, size_t workspace_bytes,
                                   void* stream_) {
  CHECK(check_ptr(rope_cos, "rope_cos", true));
  CHECK(check_ptr(rope_sin, "rope_sin", true));
  return decode_attn_scores(L, batch, seq_len, q_heads, k_codes, k_scales, Khat_prev, q, rope_cos, rope_sin, score_scale,
                            scores, Khat_out, workspace, workspace_bytes, stream_, kFormDefinition);
}

}  // extern "C"

// ---- attention over a whole cache ----------------------------------------------------------------------------
namespace {
int64_t attend_pieces(int64_t tokens) { return (tokens + aquakv::kAttendPiece - 1) / aquakv::kAttendPiece; }
size_t attend_layer_bytes(int64_t pieces, int32_t q_heads) {      // sums and soft-max statistics of one layer
  return ((size_t)pieces * q_heads * (128 + 2) * sizeof(float) + 255) & ~(size_t)255;
}
constexpr size_t kAttendRoom = (size_t)32 << 20;                  // of partial results before they are merged
int check_cache(const aquakv_cache_layer* layers, int32_t n_layers, const aquakv_cache_shape* sh) {
  if (layers == nullptr || sh == nullptr) return fail(AQUAKV_ENULL, "layers / shape is NULL");
  if (n_layers < 1) return fail(AQUAKV_EINVAL, "n_layers=%d", n_layers);
  if (sh->dtype != AQUAKV_BF16 && sh->dtype != AQUAKV_FP32) return fail(AQUAKV_EINVAL, "dtype=%d", sh->dtype);
  if (sh->kv_heads < 1 || sh->kv_heads > 4096 || sh->q_heads < 1 || sh->q_heads % sh->kv_heads || sh->q_heads > 65536)
    return fail(AQUAKV_EINVAL, "q_heads=%d must be a multiple of kv_heads=%d", sh->q_heads, sh->kv_heads);
  if (sh->batch < 1 || sh->sink_rows < 0 || sh->recent_rows < 0 || sh->capacity < 0)
    return fail(AQUAKV_EINVAL, "batch=%d sink_rows=%d recent_rows=%d capacity=%lld", sh->batch, sh->sink_rows, sh->recent_rows,
                (long long)sh->capacity);
  if (sh->capacity + sh->sink_rows + sh->recent_rows > 0x7fffffff - aquakv::kAttendPiece)
    return fail(AQUAKV_EUNSUPPORTED, "capacity=%lld", (long long)sh->capacity);
  for (int32_t l = 0; l < n_layers; ++l) {
    const aquakv_layer* L = layers[l].layer;
    if (L == nullptr) continue;
    CHECK(check_layer(L));
    if (L->kv_heads != sh->kv_heads || L->dtype != sh->dtype)
      return fail(AQUAKV_EINVAL, "layer %d: kv_heads=%d dtype=%d differ from the cache's", l, L->kv_heads, L->dtype);
    // the inputs of a predictor are rows of the previous layer in `hat` (or raw_k / raw_v): kv_heads * 128 values each
    const int32_t D = L->kv_heads * L->head_dim;
    if ((L->d_in_k != 0 && L->d_in_k != D) || (L->d_in_v != 0 && L->d_in_v != 2 * D))
      return fail(AQUAKV_EINVAL, "layer %d: predictors of %d and %d inputs, a cache of %d heads needs %d and %d", l, L->d_in_k,
                  L->d_in_v, L->kv_heads, D, 2 * D);
  }
  return AQUAKV_OK;
}
size_t attend_decode_bytes(const aquakv_cache_layer* layers, int32_t n_layers, int64_t tokens) {
  size_t most = 16;
  for (int32_t l = 0; l < n_layers && tokens > 0; ++l) {
    if (layers[l].layer == nullptr) continue;
    const Plan pl = make_plan(layers[l].layer, tokens);
    most = pl.p_bytes + pl.khat_bytes > most ? pl.p_bytes + pl.khat_bytes : most;
  }
  return (most + 255) & ~(size_t)255;
}
// A third place for recovered keys: where the values of a layer and the keys of the next one are recovered in one launch, the
// attention of the layer before runs beside them and still reads its keys.  (Longer ranges: never more than those such launches take.)
size_t attend_keys_bytes(const aquakv_cache_shape* sh, int64_t tokens) {
  if (sh->dtype != AQUAKV_BF16 || tokens <= 0) return 0;
  const int64_t most = aquakv::fused_decode_pair_rows(sh->kv_heads * 128);
  return ((size_t)(tokens < most ? tokens : most) * sh->kv_heads * 128 * elem_bytes(sh->dtype) + 255) & ~(size_t)255;
}
// What an aquakv_attend_cache call reads and writes: nothing that it writes may lie over anything else.  Sorted once: comparing
// every pair would cost more than the launches of many layers.
int check_cache_buffers(const aquakv_cache_layer* layers, int32_t n_layers, const aquakv_cache_shape* sh, const int32_t* n_sink,
                        const int32_t* n_compressed, const int32_t* n_recent, const float* rope_cos, const float* rope_sin,
                        void* const* hat, const void* workspace, size_t workspace_used, int64_t compressed, bool adjacent) {
  const size_t row = (size_t)sh->kv_heads * 128 * elem_bytes(sh->dtype);
  const int64_t most = (int64_t)n_layers * (14 + 8) + 7;
  const std::unique_ptr<CacheRange[]> ranges(new (std::nothrow) CacheRange[most]);
  if (ranges == nullptr) return fail(AQUAKV_EINVAL, "no host memory to check %d layers", n_layers);
  int64_t n = 0, tokens = 0;
  const auto add = [&](const void* p, size_t first, size_t bytes, const char* name, int32_t layer, bool written) {
    const uintptr_t begin = reinterpret_cast<uintptr_t>(p) + first;
    if (p != nullptr && bytes != 0) ranges[n++] = {begin, begin + bytes, name, layer, written};
  };
  // rows from the first token there is to the last one, of `each` rows per sequence
  struct Span { size_t first = 0, rows = 0; };
  const auto span = [&](const int32_t* count, int64_t each) {
    Span s;
    for (int b = 0; b < sh->batch; ++b) {
      if (count[b] == 0) continue;
      if (s.rows == 0) s.first = (size_t)(b * each);
      s.rows = (size_t)(b * each + count[b]) - s.first;
    }
    return s;
  };
  const Span sink = span(n_sink, sh->sink_rows), held = span(n_compressed, sh->capacity), recent = span(n_recent, sh->recent_rows);
  for (int b = 0; b < sh->batch; ++b)
    tokens = std::max(tokens, (int64_t)n_sink[b] + n_compressed[b] + n_recent[b]);
  const size_t heads = (size_t)sh->batch * sh->q_heads * 128;
  bool hat_used[2] = {false, false};
  Params before = {};
  for (int32_t l = 0; l < n_layers; ++l) {
    const aquakv_cache_layer& c = layers[l];
    add(c.sink_k, sink.first * row, sink.rows * row, "sink_k", l, false);
    add(c.sink_v, sink.first * row, sink.rows * row, "sink_v", l, false);
    add(c.recent_k, recent.first * row, recent.rows * row, "recent_k", l, false);
    add(c.recent_v, recent.first * row, recent.rows * row, "recent_v", l, false);
    add(c.q, 0, heads * elem_bytes(sh->dtype), "q", l, false);
    add(c.out, 0, heads * sizeof(float), "out", l, true);
    if (compressed == 0) continue;
    hat_used[l & 1] |= c.layer != nullptr || !adjacent;
    if (c.layer == nullptr) {
      add(c.raw_k, held.first * row, held.rows * row, "raw_k", l, false);
      add(c.raw_v, held.first * row, held.rows * row, "raw_v", l, false);
      continue;
    }
    const size_t crow = make_plan(c.layer, 1).code_row, srow = scale_row_bytes(c.layer);
    add(c.k_codes, held.first * crow, held.rows * crow, "k_codes", l, false);
    add(c.k_scales, held.first * srow, held.rows * srow, "k_scales", l, false);
    add(c.v_codes, held.first * crow, held.rows * crow, "v_codes", l, false);
    add(c.v_scales, held.first * srow, held.rows * srow, "v_scales", l, false);
    const Params params = params_of(c.layer);
    for (int i = 0; i < 8; ++i)                              // (what a layer shares with the one before is there already)
      if (params.r[i].p != before.r[i].p || params.r[i].n != before.r[i].n) add(params.r[i].p, 0, params.r[i].n, params.r[i].name, l, false);
    before = params;
    if (adjacent) continue;
    add(c.staged_k_codes, 0, compressed * crow, "staged_k_codes", l, true);
    add(c.staged_k_scales, 0, compressed * srow, "staged_k_scales", l, true);
    add(c.staged_v_codes, 0, compressed * crow, "staged_v_codes", l, true);
    add(c.staged_v_scales, 0, compressed * srow, "staged_v_scales", l, true);
  }
  for (int i = 0; i < 4; ++i)
    if (hat_used[i >> 1]) add(hat[i], 0, compressed * row, "hat", i >> 1, true);
  add(workspace, 0, workspace_used, "workspace", 0, true);
  add(rope_cos, 0, tokens * 64 * sizeof(float), "rope_cos", 0, false);
  add(rope_sin, 0, tokens * 64 * sizeof(float), "rope_sin", 0, false);
  return check_disjoint(ranges.get(), n);
}
}  // namespace

extern "C" {

size_t aquakv_attend_cache_workspace_bytes(const aquakv_cache_layer* layers, int32_t n_layers, const aquakv_cache_shape* sh) {
  if (check_cache(layers, n_layers, sh) != AQUAKV_OK) return 0;
  const size_t one = attend_layer_bytes(sh->batch * attend_pieces(sh->sink_rows + sh->capacity + sh->recent_rows), sh->q_heads);
  const size_t fit = one < kAttendRoom ? kAttendRoom / one : 1;
  return attend_decode_bytes(layers, n_layers, sh->batch * sh->capacity) + attend_keys_bytes(sh, sh->batch * sh->capacity) +
         one * (fit < (size_t)n_layers ? fit : n_layers);
}

int aquakv_attend_cache(const aquakv_cache_layer* layers, int32_t n_layers, const aquakv_cache_shape* sh, const int32_t* n_sink,
                        const int32_t* n_compressed, const int32_t* n_recent, const float* rope_cos, const float* rope_sin,
                        float score_scale, void* const* hat, void* workspace, size_t workspace_bytes, void* stream_) {
  CHECK(check_cache(layers, n_layers, sh));
  if (n_sink == nullptr || n_compressed == nullptr || n_recent == nullptr || hat == nullptr)
    return fail(AQUAKV_ENULL, "n_sink / n_compressed / n_recent / hat is NULL");
  if ((rope_cos == nullptr) != (rope_sin == nullptr)) return fail(AQUAKV_ENULL, "rope_cos and rope_sin go together");
  CHECK(check_ptr(rope_cos, "rope_cos", false));
  CHECK(check_ptr(rope_sin, "rope_sin", false));
  const int NB = sh->batch;
  const size_t row = (size_t)sh->kv_heads * 128 * elem_bytes(sh->dtype);
  int64_t compressed = 0, pieces = 0;
  bool any_sink = false, any_recent = false;
  int first = -1, last = -1;                      // sequences with compressed tokens
  bool adjacent = true;                           // their ranges lie one behind the other as they are
  for (int b = 0; b < NB; ++b) {
    if (n_sink[b] < 0 || n_sink[b] > sh->sink_rows || n_compressed[b] < 0 || n_compressed[b] > sh->capacity || n_recent[b] < 0 ||
        n_recent[b] > sh->recent_rows)
      return fail(AQUAKV_EINVAL, "sequence %d: %d + %d + %d tokens do not fit the cache", b, n_sink[b], n_compressed[b], n_recent[b]);
    const int64_t n = (int64_t)n_sink[b] + n_compressed[b] + n_recent[b];
    if (n == 0) return fail(AQUAKV_EINVAL, "sequence %d: nothing cached", b);
    any_sink |= n_sink[b] != 0;
    any_recent |= n_recent[b] != 0;
    if (n_compressed[b] != 0) {
      if (first < 0) first = b;
      else if (last != b - 1 || n_compressed[last] != sh->capacity) adjacent = false;
      last = b;
    }
    compressed += n_compressed[b];
    pieces += attend_pieces(n);
  }
  if (pieces > 0x7fffffff / sh->kv_heads) return fail(AQUAKV_EUNSUPPORTED, "%lld pieces of the sequences", (long long)pieces);
  const size_t decode_bytes = attend_decode_bytes(layers, n_layers, compressed);
  const size_t one = attend_layer_bytes(pieces, sh->q_heads);
  CHECK(check_ptr(workspace, "workspace", true));
  if (workspace_bytes < decode_bytes + one)
    return fail(AQUAKV_EWORKSPACE, "workspace %zu B < required %zu B", workspace_bytes, decode_bytes + one);
  // keys of the layers in three places in turn, where all are recovered, few enough rows for it, and the workspace has room for the third
  bool three = sh->dtype == AQUAKV_BF16 && NB <= aquakv::kAttendSeqs && aquakv::fused_decode_pair_pays(compressed, sh->kv_heads * 128) &&
               workspace_bytes >= decode_bytes + attend_keys_bytes(sh, compressed) + one;
  for (int32_t l = 0; l < n_layers; ++l) three &= layers[l].layer != nullptr || !adjacent;
  const size_t keys_bytes = three ? attend_keys_bytes(sh, compressed) : 0;
  const size_t fit = (workspace_bytes - decode_bytes - keys_bytes) / one;
  const int hold = (int)(fit < aquakv::kAttendMergeLayers ? fit : aquakv::kAttendMergeLayers);
  for (int i = 0; i < 4; ++i) CHECK(check_ptr(hat[i], "hat", compressed != 0));
  for (int32_t l = 0; l < n_layers; ++l) {
    const aquakv_cache_layer& c = layers[l];
    CHECK(check_ptr(c.sink_k, "sink_k", any_sink));
    CHECK(check_ptr(c.sink_v, "sink_v", any_sink));
    CHECK(check_ptr(c.recent_k, "recent_k", any_recent));
    CHECK(check_ptr(c.recent_v, "recent_v", any_recent));
    CHECK(check_ptr(c.q, "q", true));
    CHECK(check_ptr(c.out, "out", true));
    if (c.layer == nullptr) {
      CHECK(check_ptr(c.raw_k, "raw_k", compressed != 0));
      CHECK(check_ptr(c.raw_v, "raw_v", compressed != 0));
    } else if (compressed != 0) {
      CHECK(check_ptr(c.k_codes, "k_codes", true));
      CHECK(check_scales(c.layer, c.k_scales, "k_scales", true));
      CHECK(check_ptr(c.v_codes, "v_codes", true));
      CHECK(check_scales(c.layer, c.v_scales, "v_scales", true));
      if (!adjacent) {
        CHECK(check_ptr(c.staged_k_codes, "staged_k_codes", true));
        CHECK(check_scales(c.layer, c.staged_k_scales, "staged_k_scales", true));
        CHECK(check_ptr(c.staged_v_codes, "staged_v_codes", true));
        CHECK(check_scales(c.layer, c.staged_v_scales, "staged_v_scales", true));
      }
    }
  }
  if (compressed != 0 && layers[0].layer != nullptr && (layers[0].layer->d_in_k != 0 || layers[0].layer->d_in_v != 0))
    return fail(AQUAKV_ENULL, "layer 0 has predictors, but no layer comes before it");
  CHECK(check_cache_buffers(layers, n_layers, sh, n_sink, n_compressed, n_recent, rope_cos, rope_sin, hat, workspace,
                            decode_bytes + keys_bytes + one * (size_t)(hold < n_layers ? hold : n_layers), compressed, adjacent));
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  const int64_t first_row = first * sh->capacity;

  // the ranges of the sequences one behind the other
  aquakv::CopyRange copies[aquakv::kCopyRangesPerLaunch];        // one launch's worth at a time: nothing is allocated here
  int n_copies = 0;
  const auto send = [&]() {
    const int n = n_copies;
    n_copies = 0;
    return n == 0 ? hipSuccess : aquakv::launch_copy_ranges(copies, n, stream);
  };
  const auto gather = [&](void* dst, const void* src, size_t row_bytes) {
    int64_t to = 0;
    for (int b = first; b <= last; ++b) {
      if (n_compressed[b] == 0) continue;
      if (n_copies == aquakv::kCopyRangesPerLaunch)
        if (const hipError_t e = send()) return e;
      copies[n_copies++] = {at(dst, to, row_bytes), at(src, b * sh->capacity, row_bytes), n_compressed[b] * row_bytes};
      to += n_compressed[b];
    }
    return hipSuccess;
  };
  if (compressed != 0 && !adjacent) {
    for (int32_t l = 0; l < n_layers; ++l) {
      const aquakv_cache_layer& c = layers[l];
      if (c.layer == nullptr) continue;
      const size_t crow = make_plan(c.layer, 1).code_row, srow = scale_row_bytes(c.layer);
      HIP_TRY(gather(c.staged_k_codes, c.k_codes, crow));
      HIP_TRY(gather(c.staged_k_scales, c.k_scales, srow));
      HIP_TRY(gather(c.staged_v_codes, c.v_codes, crow));
      HIP_TRY(gather(c.staged_v_scales, c.v_scales, srow));
    }
    HIP_TRY(send());
  }
  float* const part = reinterpret_cast<float*>(static_cast<unsigned char*>(workspace) + decode_bytes + keys_bytes);
  const int64_t part_elems = pieces * sh->q_heads * 128, layer_elems = (int64_t)(one / sizeof(float));
  // where layer l's codes and scales are read (k_codes, k_scales, v_codes, v_scales), and its recovered tensors go
  struct Coded { const uint8_t* k_codes; const uint16_t* k_scales; const uint8_t* v_codes; const uint16_t* v_scales; };
  const auto coded_at = [&](int32_t l) {
    const aquakv_cache_layer& c = layers[l];
    if (!adjacent) return Coded{c.staged_k_codes, c.staged_k_scales, c.staged_v_codes, c.staged_v_scales};
    const size_t crow = make_plan(c.layer, 1).code_row, srow = scale_row_bytes(c.layer);
    return Coded{static_cast<const uint8_t*>(at(c.k_codes, first_row, crow)), static_cast<const uint16_t*>(at(c.k_scales, first_row, srow)),
                 static_cast<const uint8_t*>(at(c.v_codes, first_row, crow)), static_cast<const uint16_t*>(at(c.v_scales, first_row, srow))};
  };
  // The keys of a layer need the keys before, not its values: where a launch for one tensor leaves CUs idle, the values of layer l
  // and the keys of layer l + 1 are recovered together.  The last two layers' keys end in their own places of `hat` either way.
  const int D = sh->kv_heads * 128;
  const auto keys_at = [&](int32_t l) {
    const int from_end = (n_layers - 1 - l) % 3;
    if (!three) return hat[2 * (l & 1)];
    return from_end == 2 ? static_cast<void*>(static_cast<unsigned char*>(workspace) + decode_bytes) : hat[2 * ((n_layers - 1 - from_end) & 1)];
  };
  const auto with_next = [&](int32_t l) {
    const aquakv_layer *a = layers[l].layer, *b = l + 1 < n_layers ? layers[l + 1].layer : nullptr;
    return a != nullptr && b != nullptr && a->dtype == AQUAKV_BF16 && a->d_in_v != 0 && b->d_in_k != 0 && quantizer_id(a) == quantizer_id(b) &&
           is_wide(a) == is_wide(b) && aquakv::fused_decode_pair_pays(compressed, D);
  };
  const auto key_tensor = [&](int32_t l, const void* Kp, void* K) {
    const aquakv_layer* const L = layers[l].layer;
    const Coded in = coded_at(l);
    return aquakv::FusedTensor{Kp, nullptr, L->d_in_k, 0, L->w_k, L->b_k, L->signs_k, nullptr, const_cast<uint8_t*>(in.k_codes),
                               const_cast<uint16_t*>(in.k_scales), K};
  };
  const auto value_tensor = [&](int32_t l, const void* Vp, const void* K, void* V) {
    const aquakv_layer* const L = layers[l].layer;
    const Coded in = coded_at(l);
    return aquakv::FusedTensor{Vp, K, D, D, L->w_v, L->b_v, L->signs_v, nullptr, const_cast<uint8_t*>(in.v_codes),
                               const_cast<uint16_t*>(in.v_scales), V};
  };
  // The attention of a layer is not launched at once: it needs nothing of the next layer, and runs beside that one's recovery on the CUs
  // that the tiles leave idle: beside values and next keys in one launch, or beside the keys (beside the values, whose launch takes
  // longer, four sequences of 1800 tokens and 8 layers take 0.983 of the time of attention by itself, beside the keys 0.963).
  // `waiting`: that of the layer before (only one launch's worth of sequences can wait).
  aquakv::AttendCacheArgs waiting = {};
  bool is_waiting = false;
  int held = 0, done = 0;                                        // layers with partial results, and before them
  const auto set_sequences = [&](int b0, aquakv::AttendCacheArgs& a, int64_t& from, int& piece) {
    a.seq0 = b0;
    a.pieces.n_seq = NB - b0 < aquakv::kAttendSeqs ? NB - b0 : aquakv::kAttendSeqs;
    for (int i = 0; i < a.pieces.n_seq; ++i) {
      const int b = b0 + i;
      a.pieces.first[i] = piece;
      a.n_sink[i] = n_sink[b]; a.n_compressed[i] = n_compressed[b];
      a.n_tokens[i] = n_sink[b] + n_compressed[b] + n_recent[b];
      a.compressed_row[i] = from;
      from += n_compressed[b];
      piece += (int)attend_pieces(a.n_tokens[i]);
    }
    a.pieces.first[a.pieces.n_seq] = piece;
  };
  // the layers held are merged once their partial results fill the room, or are the last
  const auto merge = [&](const aquakv::AttendCacheArgs& a) {
    aquakv::MergeArgs m = {};
    m.part = part; m.stats = part + part_elems;
    m.part_layer = m.stats_layer = layer_elems;
    m.q_heads = sh->q_heads; m.seq0 = a.seq0; m.pieces = a.pieces;
    for (int i = 0; i < held; ++i) m.out[i] = layers[done + i].out;
    return aquakv::launch_merge_pieces(m, held, stream);
  };
  const auto merge_due = [&] { return held == hold || done + held == n_layers; };
  const auto merged = [&] { done += held; held = 0; };
  const auto attended = [&]() {                                  // `waiting` has been launched
    is_waiting = false;
    if (!merge_due()) return hipSuccess;
    const hipError_t e = merge(waiting);
    merged();
    return e;
  };
  const auto attend_now = [&]() {
    if (!is_waiting) return hipSuccess;
    if (const hipError_t e = aquakv::launch_attend_cache(sh->dtype, waiting, stream)) return e;
    return attended();
  };
  // n = 1 or 2 tensors on tiles, with the attention that waits if there is one
  const auto decode_tiles = [&](const aquakv_layer* L, const aquakv::FusedTensor* t, const float* const* codebooks, int n) {
    const aquakv::AttendCacheArgs none = {};
    const hipError_t e = aquakv::launch_fused_decode_attend(quantizer_id(L), t, codebooks, n, compressed, D, is_wide(L),
                                                            is_waiting ? waiting : none, stream);
    return e != hipSuccess || !is_waiting ? e : attended();
  };
  const auto takes_attention = [&](const aquakv_layer* L, int32_t d_in) {
    return is_waiting && L->dtype == AQUAKV_BF16 && d_in != 0 && aquakv::fused_decode_attend_fits(compressed, D);
  };
  const void *Kp = nullptr, *Vp = nullptr;
  bool have_keys = false;                                        // of this layer, from the launch of the one before
  for (int32_t l = 0; l < n_layers; ++l) {
    const aquakv_cache_layer& c = layers[l];
    void *K = keys_at(l), *V = hat[2 * (l & 1) + 1];
    if (compressed != 0 && c.layer != nullptr) {
      const Coded in = coded_at(l);
      const bool pair = with_next(l);
      if (!have_keys) {
        if (takes_attention(c.layer, c.layer->d_in_k) && !(pair && three)) {
          const aquakv::FusedTensor k = key_tensor(l, Kp, K);
          HIP_TRY(decode_tiles(c.layer, &k, &c.layer->codebook, 1));
          have_keys = true;
        } else if (pair) {
          CHECK(aquakv_decode_layer(c.layer, compressed, in.k_codes, in.k_scales, nullptr, nullptr, Kp, nullptr, K, nullptr, workspace,
                                    decode_bytes, stream));
          have_keys = true;
        } else {
          HIP_TRY(attend_now());
          CHECK(aquakv_decode_layer(c.layer, compressed, in.k_codes, in.k_scales, in.v_codes, in.v_scales, Kp, Vp, K, V, workspace,
                                    decode_bytes, stream));
        }
      }
      if (pair) {
        if (!three) HIP_TRY(attend_now());                       // (the keys it reads are about to be overwritten)
        const aquakv::FusedTensor t[2] = {value_tensor(l, Vp, K, V), key_tensor(l + 1, K, keys_at(l + 1))};
        const float* const codebooks[2] = {c.layer->codebook, layers[l + 1].layer->codebook};
        HIP_TRY(decode_tiles(c.layer, t, codebooks, 2));
      } else if (have_keys && takes_attention(c.layer, c.layer->d_in_v)) {
        const aquakv::FusedTensor v = value_tensor(l, Vp, K, V);
        HIP_TRY(decode_tiles(c.layer, &v, &c.layer->codebook, 1));
      } else if (have_keys) {
        CHECK(aquakv_decode_values(c.layer, compressed, in.v_codes, in.v_scales, Vp, K, V, workspace, decode_bytes, stream));
      }
      have_keys = pair;
      Kp = K; Vp = V;
    } else if (compressed != 0 && adjacent) {
      Kp = at(c.raw_k, first_row, row); Vp = at(c.raw_v, first_row, row);
    } else if (compressed != 0) {
      HIP_TRY(gather(K, c.raw_k, row));
      HIP_TRY(gather(V, c.raw_v, row));
      HIP_TRY(send());
      Kp = K; Vp = V;
    }
    HIP_TRY(attend_now());
    aquakv::AttendCacheArgs a = {};
    a.sink_k = c.sink_k; a.sink_v = c.sink_v; a.compressed_k = Kp; a.compressed_v = Vp; a.recent_k = c.recent_k; a.recent_v = c.recent_v;
    a.q = c.q; a.rope_cos = rope_cos; a.rope_sin = rope_sin;
    a.part = part + held * layer_elems; a.stats = a.part + part_elems;
    a.scale = score_scale;
    a.kv_heads = sh->kv_heads; a.q_heads = sh->q_heads; a.sink_rows = sh->sink_rows; a.recent_rows = sh->recent_rows;
    ++held;
    int64_t from = 0;
    int piece = 0;
    if (NB <= aquakv::kAttendSeqs) {
      set_sequences(0, a, from, piece);
      waiting = a;
      is_waiting = true;
      if (l + 1 == n_layers) HIP_TRY(attend_now());
      continue;
    }
    for (int b0 = 0; b0 < NB; b0 += aquakv::kAttendSeqs) {
      set_sequences(b0, a, from, piece);
      HIP_TRY(aquakv::launch_attend_cache(sh->dtype, a, stream));
      if (merge_due()) HIP_TRY(merge(a));
    }
    if (merge_due()) merged();
  }
  return AQUAKV_OK;
}

}  // extern "C"

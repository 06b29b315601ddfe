// Host-side launchers of the gfx950 kernels (one per stage).  Arguments are
// validated by the C-ABI layer before these are called.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace aquakv {

enum Dtype : int { kBF16 = 0, kFP32 = 1 };

// P[T, D] = [x0 (T x d0) | x1 (T x d1)] W^T + bias, W is [D, d0 + d1] row-major.
hipError_t launch_predict(int dtype, const void* x0, int d0, const void* x1, int d1, const void* W,
                          const float* bias, float* P, int64_t T, int D, hipStream_t stream);

// One tensor of a quantize / dequantize launch; rows of H heads of 128.
struct QuantizeIo {
  const void* X;              // quantize: the values
  const int8_t* signs;
  uint8_t* codes;             // written by quantize, read by dequantize
  uint16_t* scales;
  void* Xhat;                 // reconstruction (quantize: nullable)
};
// fp32 predictions [T, D], row t: outputs [0, split) at first + t * stride and the others at second + t * stride.  (Groups across
// the heads keep them in two halves, one of them in the rows of Xhat that the quantizer will write: contiguous() is the plain form.)
struct Prediction {
  float *first, *second;
  int64_t stride;
  int split;
  static Prediction contiguous(const float* P, int D) {
    return {const_cast<float*>(P), const_cast<float*>(P) + D / 2, D, D / 2};
  }
};
// Q(X - P): codes, scales and (optionally) the reconstruction of io[0 .. tensors - 1] (1 or 2, P likewise, in one layout), T rows each.
// wide: rotation groups of 1024 = the whole token (H must be 8), scales [T] instead of [T, H].
// `table` (nullable): nearest-grid-point search table from launch_build_search_table.
// wide: P may share its rows with Xhat (2 T D bytes of it, in the halves form): a wave reads its token's before it writes it.
hipError_t launch_quantize(int dtype, int n_codewords, const QuantizeIo* io, int tensors, const Prediction* P,
                           const float* codebook, const void* table, int64_t T, int H, bool wide, hipStream_t stream);

// 64 x 64 cells x 4 candidate bytes = 16 KiB, and 128 overflow lists of 8 candidate bytes.
constexpr size_t kSearchTableBytes = (64 * 64 + 2 * 128) * 4;     // cell entries + overflow lists (codec_core.h)
hipError_t launch_build_search_table(const float* codebook, int n_codewords, void* table, hipStream_t stream);

hipError_t launch_dequantize(int dtype, int n_codewords, const QuantizeIo* io, int tensors, const float* P,
                             const float* codebook, int64_t T, int H, bool wide, hipStream_t stream);

// scores[b, qh, t] for rows [row0, row0 + rows) of the flattened [batch*seq_len] axis.
// codes/scales/P/Khat_out point at row `row0`; q and scores at their tensor bases.
// rope_cos / rope_sin (nullable, fp32 [seq_len, 64]): rotate the decoded key of token t by position t first.
hipError_t launch_attn_scores(int dtype, int n_codewords, const uint8_t* codes, const uint16_t* scales, const float* P,
                              const int8_t* signs, const float* codebook, const void* q, float score_scale,
                              float* scores, void* Khat_out, int64_t row0, int64_t rows, int seq_len, int H,
                              int q_heads, const float* rope_cos, const float* rope_sin, bool wide, hipStream_t stream);

// Fused bf16 forms: prediction [x0 | x1] W^T + bias on the matrix cores, consumed in the same
// kernel by the quantizer (encode), its inverse (decode) or its inverse plus q.k (scores).
// wide (decode, scores, weighted; D = 1024): rotation groups of 1024 = the whole token, one scale per token.
hipError_t launch_fused_encode(int n_codewords, const void* x0, int d0, const void* x1, int d1, const void* W,
                               const float* bias, const int8_t* signs, const float* codebook, const void* table,
                               const void* X, uint8_t* codes, uint16_t* scales, void* Xhat, int64_t T, int D,
                               hipStream_t stream);
// The prediction of launch_predict (bf16, same bits) on whichever tiles of the fused forms suit the number of rows; P.split a multiple
// of 256 (D a multiple of 256) or of 128.
hipError_t launch_tile_predict(const void* x0, int d0, const void* x1, int d1, const void* W, const float* bias, const Prediction& P,
                               int64_t T, int D, hipStream_t stream);
// The encoder for rotation groups of 1024 (8 heads): a workgroup owns 64 tokens x all heads.  `w_retiled`: device scratch of
// 1024 * (d0 + d1) * 2 bytes, 16-byte aligned, that the call fills with the weights in the order its main loop reads them.
hipError_t launch_fused_encode_wide(int n_codewords, const void* x0, int d0, const void* x1, int d1, const void* W,
                                    void* w_retiled, const float* bias, const int8_t* signs, const float* codebook,
                                    const void* table, const void* X, uint8_t* codes, uint16_t* scales, void* Xhat,
                                    int64_t T, int D, hipStream_t stream);
hipError_t launch_fused_decode(int n_codewords, const void* x0, int d0, const void* x1, int d1, const void* W,
                               const float* bias, const int8_t* signs, const float* codebook, const uint8_t* codes,
                               const uint16_t* scales, void* Xhat, int64_t T, int D, bool wide, hipStream_t stream);
hipError_t launch_fused_scores(int n_codewords, const void* x0, int d0, const void* W, const float* bias,
                               const int8_t* signs, const float* codebook, const uint8_t* codes,
                               const uint16_t* scales, const void* q, float score_scale, float* scores, void* Khat_out,
                               int seq_len, int q_heads, int64_t T, int D, const float* rope_cos, const float* rope_sin,
                               bool wide, hipStream_t stream);

// Keys and values of a layer of few rows (fused_layer_fits) in two launches of the fused forms.  The values' predictor reads
// [Vhat_prev | Khat], and the half of its product that needs no keys runs beside the keys' launch, on CUs that launch leaves idle;
// the values' launch goes on from its fp32 sums.  Those wait in the values' Xhat and in `sums`, 16 bits of each in either (T * D * 2
// bytes), so values.Xhat is required and may not be values.X; a tile reads its share of them before it writes its rows.  Same order
// of the sums, same bits.
// Encode of 128 tokens (keys and values) 20.8 -> 18.7 us, 300 tokens at 4 bits 25.1 -> 23.7, decode of 300 tokens 17.0 -> 16.3.
struct FusedTensor {
  const void *x0, *x1;        // predictor inputs, d0 and d1 wide (keys: d1 = 0; values: x1 = the keys' Xhat)
  int d0, d1;
  const void* W;
  const float* bias;
  const int8_t* signs;
  const void* X;              // encode
  uint8_t* codes;
  uint16_t* scales;
  void* Xhat;
};
bool fused_layer_fits(int64_t T, int D);
hipError_t launch_fused_layer(bool encode, int n_codewords, const float* codebook, const void* table, const FusedTensor& keys,
                              const FusedTensor& values, void* sums, int64_t T, int D, bool wide, hipStream_t stream);
// Values of one layer and keys of the next one (which need nothing of those values), of one quantizer (bf16).
// Decode of both in one launch where it pays:
bool fused_decode_pair_pays(int64_t T, int D);
int64_t fused_decode_pair_rows(int D);      // the most rows for which it does
// Decode of n = 1 or 2 (where fused_decode_pair_pays) tensors, with attention over a layer recovered before on the CUs that it
// leaves idle or free early (no pieces: none).  n = 1: where fused_decode_attend_fits.
struct AttendCacheArgs;
bool fused_decode_attend_fits(int64_t T, int D);
hipError_t launch_fused_decode_attend(int n_codewords, const FusedTensor* tensors, const float* const* codebooks, int n, int64_t T, int D,
                                      bool wide, const AttendCacheArgs& attend, hipStream_t stream);
// Encode of both, fused with the quantizer in one launch where it pays, with tables and codebooks of their own:
bool fused_encode_pair_pays(int64_t T, int D);
hipError_t launch_fused_encode_pair(int n_codewords, const FusedTensor* tensors, const float* const* codebooks, const void* const* tables,
                                    int64_t T, int D, hipStream_t stream);
// The predictions of both in one launch (`out` as in launch_tile_predict), of up to tile_predict_pair_rows() rows:
int64_t tile_predict_pair_rows(int D);
hipError_t launch_tile_predict_pair(const FusedTensor* tensors, const Prediction* out, int64_t T, int D, hipStream_t stream);

// The same on tiles of 256 tokens x two heads (D a multiple of 256; wide: decode only): same bits, a faster main
// loop, half as many workgroups.  launch_fused_encode / _decode / _scores take this form by themselves for ranges that
// fill the chip more than once (below that: fused_tile.h) when two_heads_pays(T, D): when the larger tile costs no extra
// round over the CUs.
bool two_heads_pays(int64_t T, int D);
hipError_t launch_predict_two_heads(const void* x0, int d0, const void* x1, int d1, const void* W, const float* bias, const Prediction& P,
                                    int64_t T, int D, hipStream_t stream);
hipError_t launch_fused_encode_two_heads(int n_codewords, const void* x0, int d0, const void* x1, int d1, const void* W,
                                         const float* bias, const int8_t* signs, const float* codebook, const void* table,
                                         const void* X, uint8_t* codes, uint16_t* scales, void* Xhat, int64_t T, int D,
                                         hipStream_t stream);
hipError_t launch_fused_decode_two_heads(int n_codewords, const void* x0, int d0, const void* x1, int d1, const void* W,
                                         const float* bias, const int8_t* signs, const float* codebook,
                                         const uint8_t* codes, const uint16_t* scales, void* Xhat, int64_t T, int D,
                                         bool wide, hipStream_t stream);
hipError_t launch_fused_scores_two_heads(int n_codewords, const void* x0, int d0, const void* W, const float* bias,
                                         const int8_t* signs, const float* codebook, const uint8_t* codes,
                                         const uint16_t* scales, const void* q, float score_scale, float* scores,
                                         void* Khat_out, int seq_len, int q_heads, int64_t T, int D,
                                         const float* rope_cos, const float* rope_sin, hipStream_t stream);

// Value side of attention.  The sums over tokens are taken per chunk of kWeightedChunk tokens of one sequence
// (part[batch * chunks_per_seq, q_heads, 128] fp32, chunks_per_seq = ceil(seq_len / kWeightedChunk)) and then added in
// chunk order by launch_combine_weighted: out[b, qh, :] = sum_t weights[b, qh, t] * Vhat[b * seq_len + t, qh / rep, :].
// Soft-max form (pstats given, [batch * chunks_per_seq, q_heads, 2] fp32): `weights` holds raw scores, a chunk's sums are
// taken with exp(score - chunk maximum), pstats receives that maximum and the chunk's weight sum, and the combine step
// rescales the chunks to the row maximum and divides by the row's weight sum (row_stats, nullable, [batch, q_heads, 2]:
// row maximum and that denominator).
constexpr int kWeightedChunk = 256;
// decode of the values with the chunk sums taken in the epilogue (bf16, seq_len a multiple of kWeightedChunk); Xhat nullable
hipError_t launch_fused_weighted(int n_codewords, const void* x0, int d0, const void* x1, int d1, const void* W,
                                 const float* bias, const int8_t* signs, const float* codebook, const uint8_t* codes,
                                 const uint16_t* scales, void* Xhat, const float* weights, float* part, float* pstats,
                                 int seq_len, int q_heads, int64_t T, int D, bool wide, hipStream_t stream);
// Chunk sums over values already decoded to memory (any dtype, any seq_len): of given weights, in soft-max form, or in soft-max form
// where a sequence is one chunk, which leaves nothing to combine: part and pstats (nullable) are out and row_stats then.
enum WeightedForm : int { kWeightedGiven = 0, kWeightedSoftMax = 1, kWeightedWhole = 2 };
hipError_t launch_weighted_values(int dtype, const void* Vhat, const float* weights, WeightedForm form, float* part, float* pstats,
                                  int batch, int seq_len, int H, int q_heads, hipStream_t stream);
hipError_t launch_combine_weighted(const float* part, const float* pstats, float* out, float* row_stats, int batch,
                                   int seq_len, int q_heads, hipStream_t stream);
// Attention of one query per sequence over `tokens` (<= kAttendRawMaxTokens) keys / values in the storage dtype
// ([batch * tokens, H, 128]), written to or merged into (accumulate != 0) out [batch, q_heads, 128] and the row
// statistics [batch, q_heads, 2] (maximum, sum of exp(score - maximum)) that launch_combine_weighted hands out.
constexpr int kAttendRawMaxTokens = 4096;
// rope_cos / rope_sin (nullable, fp32 [tokens, 64]): rotate key t by its position before the dot product.
hipError_t launch_attend_raw(int dtype, const void* K, const void* V, const void* q, const float* rope_cos,
                             const float* rope_sin, float scale, float* out, float* stats, int batch, int tokens, int H,
                             int q_heads, int accumulate, hipStream_t stream);
// probs[r, :] = softmax(scores[r, :]) for `rows` rows of length n (in place allowed)
hipError_t launch_softmax_rows(const float* scores, float* probs, int64_t rows, int64_t n, hipStream_t stream);

// Scores with the key predictor folded into the query (bf16, 8 kv heads, 1024 predictor inputs,
// q_heads <= 64): reads Khat_prev and the codes once per 4 query heads of a kv head (one pass up to 32 query
// heads, two up to 64).  `workspace`: folded_scores_workspace_bytes(batch, q_heads).
// bytes of folded query operands per batch entry and pass: u as bf16 high / low MFMA operands (8 waves x 2 x 8 k
// steps x 1 KiB), the rotated queries [32][128] fp32, q . b [32] fp32
constexpr size_t kFoldedBytesPerBatch = (size_t)8 * 2 * 8 * 1024 + 32 * 128 * 4 + 32 * 4;
bool folded_scores_supported(int kv_heads, int d_in_k, int q_heads);
size_t folded_scores_workspace_bytes(int batch, int q_heads);
hipError_t launch_folded_scores(int n_codewords, const void* Khat_prev, const void* W, const float* bias,
                                const int8_t* signs, const float* codebook, const uint8_t* codes,
                                const uint16_t* scales, const void* q, float score_scale, float* scores, void* workspace,
                                int batch, int seq_len, int q_heads, hipStream_t stream);

// Attention over the caches of up to kAttendSeqs sequences (attend_cache.hip).  Sequence b of the launch has pieces
// [first[b], first[b + 1]) of kAttendPiece tokens each, numbered over the whole batch.
constexpr int kAttendPiece = 64;
constexpr int kAttendSeqs = 64;                   // sequences per launch: their counts travel in the kernel arguments
constexpr int kAttendMergeLayers = 32;            // layers merged per launch
struct Pieces {
  int n_seq;
  int first[kAttendSeqs + 1];
};
struct AttendCacheArgs {
  const void *sink_k, *sink_v, *compressed_k, *compressed_v, *recent_k, *recent_v;    // rows of kv_heads x 128
  const void* q;                                  // [batch, q_heads, 128]
  const float *rope_cos, *rope_sin;               // nullable, [tokens, 64]
  float *part, *stats;                            // [pieces, q_heads, 128], [pieces, q_heads, 2]
  float scale;
  int kv_heads, q_heads, sink_rows, recent_rows;  // rows per sequence of the sink and recent tensors
  int64_t seq0;                                   // the launch's first sequence
  int n_sink[kAttendSeqs], n_compressed[kAttendSeqs], n_tokens[kAttendSeqs];
  int64_t compressed_row[kAttendSeqs];            // first row of a sequence's compressed range
  Pieces pieces;
};
hipError_t launch_attend_cache(int dtype, const AttendCacheArgs& a, hipStream_t stream);
struct MergeArgs {
  const float *part, *stats;
  int64_t part_layer, stats_layer;                // elements from one layer to the next
  int q_heads;
  int64_t seq0;
  float* out[kAttendMergeLayers];
  Pieces pieces;
};
hipError_t launch_merge_pieces(const MergeArgs& a, int layers, hipStream_t stream);

// Ridge least-squares fit of a predictor, W [d_out, d0 + d1] = argmin || [x0 | x1] W^T - Y ||^2 + lambda ||W||^2 with
// lambda = rate * trace(X^T X) / d_in, in fp64 through the normal equations.  d0, d1, d_out multiples of 64.
// `workspace`: fit_workspace_bytes(d0 + d1, d_out).  W64 (nullable): the unrounded solution [d_out, d_in].
// bias (nullable, fp32 [d_out]): fit an intercept as well (centred regression).
size_t fit_workspace_bytes(int d_in, int d_out);
hipError_t launch_fit_predictor(int dtype, int64_t tokens, const void* x0, int d0, const void* x1, int d1, const void* Y,
                                int d_out, double rate, void* W, double* W64, float* bias, void* workspace,
                                hipStream_t stream);

// The Gram products of a fit over bf16 data in integers (exact_gram.hip): blocks of G [d0 + d1 + d_out, d0 + d1] on and below the diagonal, the
// others are scratch.  G, flag and 8 bytes per column of [x0 | x1 | Y] at `columns` are zero before.  flag != 0 after: G's blocks on and below
// the diagonal are still zero.
bool exact_gram_fits(int64_t tokens, int d0, int d1, int d_out);
hipError_t launch_exact_gram(int64_t tokens, const void* x0, int d0, const void* x1, int d1, const void* Y, int d_out, double* G, void* columns,
                             int* flag, hipStream_t stream);

// Device-to-device copies of n byte ranges, kCopyRangesPerLaunch per launch (3 KiB of kernel arguments).
struct CopyRange { void* dst; const void* src; size_t bytes; };
constexpr int kCopyRangesPerLaunch = 128;
hipError_t launch_copy_ranges(const CopyRange* ranges, int n, hipStream_t stream);

}  // namespace aquakv

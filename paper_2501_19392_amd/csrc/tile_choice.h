// Which tile a launch of the fused predictor kernels takes.  Host code only, no HIP.
#pragma once
#include <cstdint>
#include <initializer_list>

namespace aquakv {

// Rows per tile (fused_tile.h) of a launch over n_seq sequences of seq_len rows (one sequence for encode and decode);
// 0: the tiles of 256 rows x one or two heads.
//
// A CU holds one workgroup, so what counts is the rounds of workgroups over the CUs and the rows of a round.  Ranges that
// fill the chip in one round take the smallest tile that still does.  Keys and values x 8 heads, us (with main loops whose waves all loaded and
// multiplied; now a tenth less, and no size between 3100 and 6144 tokens has a tile more than 2 % faster than its own):
//   1024 tokens  encode 23.6 on 32 rows, 27.0 on 64, 38.8 on 128 (decode 19.1, 22.3, 30.7)
//   2048         28.7 on 64, 39.5 on 128 (24.3, 31.1)
//   2100         34.1 on 96, 39.8 on 128 (28.7, 31.4); 3072 39.2, 41.9 (32.4, 32.7)
//   4096         a tensor at a time 20.6 / 28.8 on 128, 26.1 / 35 on 256
//   4200         55.1 on 192, 59.4 on 256 (44.4, 44.7); 6144 61.9, 66.2 (51.5, 50.8); groups across the heads, whose predictions have a large
//                tile of two heads, 76.6, 98.0 (49.6, 52.9) and 86.0, 101.4 (57.1, 58.6)
// The scoring calls gain on all of them, a sequence or many: 2600 tokens with the rotary embedding 13.7 on 96, 15.5 on 128, 32 x 96 14.8, 15.8, 4 x 700
// 14.4, 14.9; 4200 tokens 21.0 on 192, 23.6 on 256, 6144 24.1, 25.1, 4 x 1300 22.8, 26.5, 16 x 384 24.5, 27.0; groups across the heads 5 to 20 %.
//
// Beyond that a launch takes several rounds, and the tile is the one whose rounds cost least.  What a round costs, us of an encode of keys and values
// with 16 points in a stack of layers: 66 to 67 on 256 rows (9 more for the first), 122 to 126 on 256 rows x two heads, 51 to 56 on 192 rows,
// 87 to 92 on 320 rows and 100 with five rounds of them (97: above 96 the seven rounds of 256 rows are taken there).  By range, 16 points, keys and
// values, encode and decode on the tile taken / the next best:
//   8300 tokens    85 on 320 rows / 92 on 192, 64 / 69
//   10300          101 on 192 / 116 on two heads, 83 on two heads / 83; 12200 107 / 116, 84 / 83 to 91
//   16300          130 on two heads / 140 on 256, 99 / 111
//   16500          154 on 192 / 172 on 320, 121 / 129; 18400 161 / 175, 124 / 133
//   18500          175 on 320 / 190 on 192, 132 / 145
//   20600          202 on 256 / 202 on 192, 157 / 153; 24500 208 / 216, 165 / 164
//   33000          325 on 192 / 334 on 256 (256 points 371 / 399, uniform 283 / 285), 252 on 256 / 245 to 256; 36800 336 / 342 (385 / 410, 292 / 292)
//   49500          475 on 256 / 490 on 320, 364 to 378 / 380
// What differs is a round on 192 rows: 54 to encode.  Decode and scores of heads apart gain from three rounds and not surely from two or six
// (12200 tokens 91 / 87 on another card, 33000 one layer again and again 256 / 251): 63.  Across the heads two rounds pay as well where they
// decode 16 or 256 points (10300 tokens 92 / 100 and 102 / 115 on two heads, 12200 102 / 102 and 112 / 117; three rounds 159 / 188 on 320 with 256 points; six
// 322 / 324, one layer again 334 / 310) and in scores, which have no tile of two heads there (256 points 47 / 60, 53 / 62): 60.  64 points (113 / 108, 117 / 110)
// and the uniform backbone (82 / 80, 90 / 85) decode like heads apart.  Predictions alone (groups across the heads, encode) take no round on 192
// rows: 193 us against 179 at 16500 tokens.
constexpr int64_t kRound256 = 67, kFirstRound256 = 9, kRoundTwoHeads = 125, kRound320 = 97;
constexpr int64_t kEncodeRound192 = 54, kDecodeRound192 = 63, kAcrossRound192 = 60, kNoRound192 = 1 << 20;
inline int64_t decode_round_192(int n_codewords, bool across, bool scores) {
  return across && (scores || n_codewords == 16 || n_codewords == 256) ? kAcrossRound192 : kDecodeRound192;
}
inline int tile_rows(int64_t n_seq, int64_t seq_len, int D, bool two_heads, int64_t round_192) {
  constexpr int64_t kCUs = 256;                      // MI355X
  const int64_t H = D / 128;
  const auto tiles = [&](int64_t rows) { return n_seq * ((seq_len + rows - 1) / rows) * H; };
  const auto rounds = [&](int64_t t) { return (t + kCUs - 1) / kCUs; };
  for (const int rows : {32, 64, 96, 128, 192})
    if (tiles(rows) <= kCUs) return rows;
  const int64_t all = (n_seq * seq_len + 255) / 256;    // tiles of 256 rows may straddle sequences
  int64_t other = kRound256 * rounds(all * H) + kFirstRound256;
  if (two_heads && D % 256 == 0 && kRoundTwoHeads * rounds(all * H / 2) < other) other = kRoundTwoHeads * rounds(all * H / 2);
  const int64_t on_320 = kRound320 * rounds(tiles(320)), on_192 = round_192 * rounds(tiles(192));
  if (on_192 < on_320 && on_192 < other) return 192;
  return on_320 < other ? 320 : 0;
}

}  // namespace aquakv

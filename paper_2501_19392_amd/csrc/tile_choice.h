// Which tile a launch of the fused predictor kernels takes.  Host code only, no HIP.
#pragma once
#include <cstdint>
#include <initializer_list>

namespace aquakv {

// Rows per tile (fused_tile.h) of a launch over n_seq sequences of seq_len rows (one sequence for encode and decode);
// 0: the tiles of 256 rows x one or two heads.
//
// A CU holds one workgroup, so what counts is the rounds of workgroups over the CUs and the rows of a round.  Ranges that
// fill the chip in one round take the smallest tile that still does.  Keys and values x 8 heads, a stack of layers, us a layer:
//   1024 tokens  encode 21.2 on 32 rows, 23.2 on 64, 32.7 on 128 (decode 17.3, 18.6, 24.5)
//   2048         25.5 on 64, 28.0 on 96, 33.7 on 128 (20.7, 22.3, 25.5)
//   2100         28.1 on 96, 33.9 on 128 (22.4, 25.6); 3072 30.6, 35.2 (24.8, 26.8)
//   4096         39.1 on 128, 44.1 on 192, 54.1 on 256 (30.2, 33.3, 39.6)
//   4200         43.8 on 192, 54.3 on 256 (33.4, 40.0); 6144 50.2, 59.2 (39.5, 44.4)
// Scores: 2600 tokens 10.3 on 96, 11.4 on 128, 4200 16.0 on 192, 19.5 on 256, 6144 18.2, 21.3; with groups across the heads 11.5, 13.4; 18.3, 23.0;
// 20.6, 24.7.
//
// Beyond that a launch takes several rounds, and the tile is the one whose rounds cost least.  What a round costs, us of an encode of keys and values
// with 16 points in a stack of layers: 66 to 67 on 256 rows (9 more for the first), 122 to 126 on 256 rows x two heads, 51 to 56 on 192 rows,
// 87 to 92 on 320 rows and 100 with five rounds of them (97: above 96 the seven rounds of 256 rows are taken there).  By range, 16 points, keys and
// values, encode and decode on the tile taken / the next best:
//   8300 tokens    85 on 320 rows / 92 on 192, 64 / 69
//   10300          101 on 192 / 116 on two heads (uniform 98 on two heads / 93), 83 on two heads / 83; 12200 107 / 116, 84 / 83 to 91
//   16300          130 on two heads / 140 on 256, 99 / 111
//   16500          154 on 192 / 172 on 320, 121 / 129; 18400 161 / 175, 124 / 133
//   18500          175 on 320 / 190 on 192, 132 / 145
//   20600          202 on 256 / 202 on 192, 157 / 153; 24500 208 / 216, 165 / 164
//   33000          325 on 192 / 334 on 256 (256 points 371 / 399), 252 on 256 / 245 to 256; 36800 336 / 342 (385 / 410)
//   49500          475 on 256 / 490 on 320, 364 to 378 / 380
// What differs is a round on 192 rows: 54 to encode with a grid.  Elsewhere three rounds gain (across the heads with 256 points 159 / 188 on 320 rows at
// 16500 tokens, one layer on changing buffers 170 / 192) and two or six not surely: 63.  Two rounds against one of two heads, in a stack / one layer on three
// sets of buffers in turn: uniform encode of 11000 tokens 95 to 98 / 100 to 97, decode of 10800 across the heads with 256 points 107 to 115 / 113 to 108;
// six against five of 256 rows, decode of 33000 tokens 245 to 252 / 256 to 251.  Scores across the heads have no tile of two heads, and take two
// rounds as well (10300 tokens, 256 points, 47 / 60 on 256 rows, 12200 52 / 62).  Predictions alone (groups across the heads, encode) take none of several rounds
// on 192 rows: 193 us against 179 at 16500 tokens.
constexpr int64_t kRound256 = 67, kFirstRound256 = 9, kRoundTwoHeads = 125, kRound320 = 97;
constexpr int64_t kSearchRound192 = 54, kRound192 = 63, kNoRound192 = 1 << 20;
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

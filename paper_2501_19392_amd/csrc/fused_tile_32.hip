// Fused predictor kernels on tiles of 32 token rows x one kv head (fused_tile.h).
#include "fused_tile.h"

namespace aquakv {

AQUAKV_TILE_LAUNCHER(32) { return launch_tile<1>(mode, n_codewords, wide, n_seq, a, stream); }

AQUAKV_TILE_ATTEND_LAUNCHER(32) { return launch_tile_attend<1>(n_codewords, wide, jobs, n, attend, stream); }

hipError_t launch_pair_32(int mode, int n_codewords, bool wide, const TileArgs& a, const TileArgs& b, hipStream_t stream) {
  TilePair pair;
  const TileArgs jobs[2] = {a, b};
  const unsigned blocks = (unsigned)pair_jobs<1>(pair, jobs, 2);
#define AQUAKV_TILE(N, MODE, WIDE) fused_tile_pair_kernel<N, MODE, WIDE><<<blocks, Tile<1>::kThreads, 0, stream>>>(pair)
  if (mode == kTileEncode && !wide) AQUAKV_TILE_N(kTileEncode, false);
  else if (mode == kTileDecode && wide) AQUAKV_TILE_N(kTileDecode, true);
  else if (mode == kTileDecode) AQUAKV_TILE_N(kTileDecode, false);
  else return hipErrorInvalidValue;
#undef AQUAKV_TILE
  return hipGetLastError();
}

hipError_t launch_tile_rest(int mode, int n_codewords, bool wide, const TileArgs& args, hipStream_t stream) {
  using S = Tile<1>;
  TileArgs a = args;
  a.tiles_per_seq = (a.seq_len + S::kRows - 1) / S::kRows;
  a.xcd = xcd_split(a.tiles_per_seq, a.D / kGroup, S::kRows);
  const unsigned blocks = (unsigned)(a.tiles_per_seq * (a.D / kGroup));
#define AQUAKV_TILE(N, MODE, WIDE) fused_tile_kernel<N, MODE, 1, WIDE, kUseSums><<<blocks, S::kThreads, 0, stream>>>(a)
  if (mode == kTileEncode && !wide) AQUAKV_TILE_N(kTileEncode, false);
  else if (mode == kTileDecode && wide) AQUAKV_TILE_N(kTileDecode, true);
  else if (mode == kTileDecode) AQUAKV_TILE_N(kTileDecode, false);
  else return hipErrorInvalidValue;
#undef AQUAKV_TILE
  return hipGetLastError();
}

AQUAKV_TILE_TWO_LAUNCHER(32) { return launch_tile_two<1>(mode, n_codewords, jobs, stream); }

}  // namespace aquakv

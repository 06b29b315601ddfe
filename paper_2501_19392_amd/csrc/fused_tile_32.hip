// Fused predictor kernels on tiles of 32 token rows x one kv head (fused_tile.h).
#include "fused_tile.h"

namespace aquakv {

AQUAKV_TILE_LAUNCHER(32) { return launch_tile<1>(mode, n_codewords, wide, n_seq, a, stream); }

hipError_t launch_tile_pair(int mode, int n_codewords, bool wide, const TileArgs& a, const TileArgs& sums, hipStream_t stream) {
  using S = Tile<1>;
  TilePair pair = {{a, sums}, 0};
  for (TileArgs& job : pair.job) job.tiles_per_seq = (job.seq_len + S::kRows - 1) / S::kRows;
  pair.blocks = pair.job[0].tiles_per_seq * (a.D / kGroup);
  const unsigned blocks = (unsigned)(pair.blocks + pair.job[1].tiles_per_seq * (sums.D / kGroup));
#define AQUAKV_TILE(N, MODE, WIDE) fused_tile_pair_kernel<N, MODE, 1, WIDE><<<blocks, S::kThreads, 0, stream>>>(pair)
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
  const unsigned blocks = (unsigned)(a.tiles_per_seq * (a.D / kGroup));
#define AQUAKV_TILE(N, MODE, WIDE) fused_tile_kernel<N, MODE, 1, WIDE, kUseSums><<<blocks, S::kThreads, 0, stream>>>(a)
  if (mode == kTileEncode && !wide) AQUAKV_TILE_N(kTileEncode, false);
  else if (mode == kTileDecode && wide) AQUAKV_TILE_N(kTileDecode, true);
  else if (mode == kTileDecode) AQUAKV_TILE_N(kTileDecode, false);
  else return hipErrorInvalidValue;
#undef AQUAKV_TILE
  return hipGetLastError();
}

}  // namespace aquakv

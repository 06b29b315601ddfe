// Fused predictor kernels on tiles of 64 token rows x one kv head (fused_tile.h).
#include "fused_tile.h"

namespace aquakv {

AQUAKV_TILE_LAUNCHER(64) { return launch_tile<2>(mode, n_codewords, wide, n_seq, a, stream); }

AQUAKV_TILE_ATTEND_LAUNCHER(64) { return launch_tile_attend<2>(n_codewords, wide, jobs, n, attend, stream); }

AQUAKV_TILE_TWO_LAUNCHER(64) { return launch_tile_two<2>(mode, n_codewords, jobs, stream); }

}  // namespace aquakv

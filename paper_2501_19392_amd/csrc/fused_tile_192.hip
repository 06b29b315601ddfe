// Fused predictor kernels on tiles of 192 token rows x one kv head (fused_tile.h).
#include "fused_tile.h"

namespace aquakv {

AQUAKV_TILE_LAUNCHER(192) { return launch_tile<6>(mode, n_codewords, wide, n_seq, a, stream); }

AQUAKV_TILE_ATTEND_LAUNCHER(192) { return launch_tile_attend<6>(n_codewords, wide, jobs, n, attend, stream); }

AQUAKV_TILE_TWO_LAUNCHER(192) { return launch_tile_two<6>(mode, n_codewords, jobs, stream); }

}  // namespace aquakv

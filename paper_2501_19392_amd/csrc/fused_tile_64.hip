// Fused predictor kernels on tiles of 64 token rows x one kv head (fused_tile.h).
#include "fused_tile.h"

namespace aquakv {

AQUAKV_TILE_LAUNCHER(64) { return launch_tile<2>(mode, n_codewords, wide, n_seq, a, stream); }

AQUAKV_PAIR_LAUNCHER(64) { return launch_pair<2>(mode, n_codewords, wide, a, b, stream); }

}  // namespace aquakv

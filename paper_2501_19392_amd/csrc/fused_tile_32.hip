// Fused predictor kernels on tiles of 32 token rows x one kv head (fused_tile.h).
#include "fused_tile.h"

namespace aquakv {

AQUAKV_TILE_LAUNCHER(32) { return launch_tile<1>(mode, n_codewords, wide, n_seq, a, stream); }

}  // namespace aquakv

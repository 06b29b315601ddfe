// Predictions of two tensors in one launch, on tiles of different sizes (fused_tile.h).
#include "fused_tile.h"

namespace aquakv {
namespace {

template <int MB0, int MB1> hipError_t launch(const TileArgs* jobs, hipStream_t stream) {
  TilePair pair;
  const unsigned blocks = (unsigned)pair_jobs<MB0, MB1>(pair, jobs, 2);
  predict_two_tiles_kernel<MB0, MB1><<<blocks, TwoTiles<MB0, MB1>::kWaves * 64, 0, stream>>>(pair);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_predict_two_tiles(int rows0, int rows1, const TileArgs* jobs, hipStream_t stream) {
  if (rows0 == 32 && rows1 == 96) return launch<1, 3>(jobs, stream);
  if (rows0 == 64 && rows1 == 128) return launch<2, 4>(jobs, stream);
  if (rows0 == 64 && rows1 == 192) return launch<2, 6>(jobs, stream);
  if (rows0 == 96 && rows1 == 192) return launch<3, 6>(jobs, stream);
  if (rows0 == 128 && rows1 == 192) return launch<4, 6>(jobs, stream);
  return hipErrorInvalidValue;
}

}  // namespace aquakv

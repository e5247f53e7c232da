// Tiled gridder: FP16 tables (see tiled_grid.h).
#include "tiled_grid.h"

namespace wproj {

hipError_t launch_tiled_grid_f16(const wproj_kernels *k, const BinShape &B, const TileShape &ts, const BinWorkspace &W,
                                 void *grid, const void *vis, hipStream_t s) {
  return dispatch_planned<float, RecordF32, half2c>(k, B, ts, W, grid, vis, s);
}

}  // namespace wproj

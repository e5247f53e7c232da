// Tiled gridder: FP64 (see tiled_grid.h).
#include "tiled_grid.h"

namespace wproj {

hipError_t launch_tiled_grid_f64(const wproj_kernels *k, const BinShape &B, const TileShape &ts, const BinWorkspace &W,
                                 void *grid, const void *vis, hipStream_t s) {
  return dispatch_planned<double, RecordF64, double2>(k, B, ts, W, grid, vis, s);
}

}  // namespace wproj

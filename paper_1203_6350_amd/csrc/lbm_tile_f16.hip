// lbm_tile_f16.hip -- tile kernels for F16 storage.
#include "lbm_tile.h"

namespace lbm {

hipError_t launch_tile_f16(const StepConfig &c, int region, int steps, const double *source,
                           const void *src, void *dst, hipStream_t stream) {
  return launch_tile_storage<__half>(c, region, steps, source, src, dst, stream);
}

hipError_t launch_batch_tile_f16(int region, int most, const BatchDomain *doms, const int4 *tiles,
                                 const int *ntiles, int grid, int j, hipStream_t stream) {
  return launch_batch_tile_storage<__half>(region, most, doms, tiles, ntiles, grid, j, stream);
}

}  // namespace lbm

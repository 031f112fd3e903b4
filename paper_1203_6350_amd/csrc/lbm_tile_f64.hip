// lbm_tile_f64.hip -- tile kernels for F64 storage.
#include "lbm_tile.h"

namespace lbm {

hipError_t launch_tile_f64(const StepConfig &c, int region, int steps, const double *source,
                           const void *src, void *dst, hipStream_t stream) {
  return launch_tile_storage<double>(c, region, steps, source, src, dst, stream);
}

}  // namespace lbm

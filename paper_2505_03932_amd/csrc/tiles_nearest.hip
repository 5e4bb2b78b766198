// Tiled forward kernels of the single image, nearest interpolation.
#include "tile_kernels.hpp"

namespace dfr {
template const void *tile_kernel_for<DFR_NEAREST>(int, int);
template const void *small_kernel_for<DFR_NEAREST>(int);
}  // namespace dfr

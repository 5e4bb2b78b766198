// Tiled forward kernels of the single image, bilinear interpolation.
#include "tile_kernels.hpp"

namespace dfr {
template const void *tile_kernel_for<DFR_BILINEAR>(int, int);
template const void *small_kernel_for<DFR_BILINEAR>(int);
}  // namespace dfr

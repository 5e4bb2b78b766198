// Tiled forward kernels of the single image, bicubic interpolation.
#include "tile_kernels.hpp"

namespace dfr {
template const void *tile_kernel_for<DFR_BICUBIC>(int, int);
template const void *small_kernel_for<DFR_BICUBIC>(int);
}  // namespace dfr

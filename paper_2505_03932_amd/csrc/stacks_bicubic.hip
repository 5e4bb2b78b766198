// Batch, cropped batch and coadd kernels, bicubic interpolation.
#include "tile_kernels.hpp"

namespace dfr {
template const void *batch_kernel_for<DFR_BICUBIC>(int, int);
template const void *coadd_kernel_for<DFR_BICUBIC>(int, int);
template const void *crop_kernel_for<DFR_BICUBIC>(int, int);
}  // namespace dfr

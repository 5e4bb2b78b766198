// Backward tile kernels, bicubic interpolation.
#include "backward_tile.hpp"

namespace dfr {
template BwdKernel bwd_pick<DFR_BICUBIC>(int, int, bool, bool);
}  // namespace dfr

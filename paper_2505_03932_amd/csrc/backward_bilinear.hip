// Backward tile kernels, bilinear interpolation.
#include "backward_tile.hpp"

namespace dfr {
template BwdKernel bwd_pick<DFR_BILINEAR>(int, int, bool, bool);
}  // namespace dfr

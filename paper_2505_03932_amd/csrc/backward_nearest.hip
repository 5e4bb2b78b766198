// Backward tile kernels, nearest interpolation.
#include "backward_tile.hpp"

namespace dfr {
template BwdKernel bwd_pick<DFR_NEAREST>(int, int, bool, bool);
}  // namespace dfr

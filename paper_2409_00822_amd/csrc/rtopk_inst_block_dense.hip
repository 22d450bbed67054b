// Instantiations: one workgroup of W wavefronts per row, for rows wider than 8192 columns and few narrower ones -- fp32 dense output.
#include "rtopk_block_kernel.hpp"

namespace rtopk {

template <int G, int NG, int W>
static hipError_t pick(int mode, const LaunchArgs& a) {
  if (mode == kExact) return launch_block<G, NG, W, kExact, false, kF32, true>(a);
  if (mode == kEarly) return launch_block<G, NG, W, kEarly, false, kF32, true>(a);
  return hipErrorInvalidValue;
}

hipError_t launch_block_dense(int g, int ng, int w, int mode, const LaunchArgs& a) {
  if (g == 4) {
    if (w == 4 && ng == 4) return pick<4, 4, 4>(mode, a);
    if (w == 4 && ng == 8) return pick<4, 8, 4>(mode, a);
    if (w == 4 && ng == 12) return pick<4, 12, 4>(mode, a);
    if (w == 4 && ng == 16) return pick<4, 16, 4>(mode, a);
    if (w == 8 && ng == 12) return pick<4, 12, 8>(mode, a);
    if (w == 8 && ng == 16) return pick<4, 16, 8>(mode, a);
    if (w == 16 && ng == 12) return pick<4, 12, 16>(mode, a);
    if (w == 16 && ng == 16) return pick<4, 16, 16>(mode, a);
    return hipErrorInvalidValue;
  }
  return hipErrorInvalidValue;
}

}  // namespace rtopk

// Instantiations: one workgroup of W wavefronts per row, for rows wider than 8192 columns and few narrower ones -- fp32 pairs: precision-bounded mode and the k smallest.
#include "rtopk_block_kernel.hpp"

namespace rtopk {

// 128-bit loads with 12 or 16 loads per lane (W = 4, 8 or 16); few rows with 4 or 8.
template <int G, int NG, int W>
static hipError_t pick(int mode, bool smallest, const LaunchArgs& a) {
  if (smallest) {
    if (mode == kExact) return launch_block<G, NG, W, kExact, true>(a);
    if (mode == kEarly) return launch_block<G, NG, W, kEarly, true>(a);
    return hipErrorInvalidValue;
  }
  if (mode == kEps) return launch_block<G, NG, W, kEps>(a);
  return hipErrorInvalidValue;
}

hipError_t launch_block_variant(int g, int ng, int w, int mode, bool smallest, const LaunchArgs& a) {
  if (g == 4) {
    if (w == 4 && ng == 4) return pick<4, 4, 4>(mode, smallest, a);
    if (w == 4 && ng == 8) return pick<4, 8, 4>(mode, smallest, a);
    if (w == 8 && ng == 4) return pick<4, 4, 8>(mode, smallest, a);
    if (w == 8 && ng == 8) return pick<4, 8, 8>(mode, smallest, a);
    if (w == 4 && ng == 12) return pick<4, 12, 4>(mode, smallest, a);
    if (w == 4 && ng == 16) return pick<4, 16, 4>(mode, smallest, a);
    if (w == 8 && ng == 12) return pick<4, 12, 8>(mode, smallest, a);
    if (w == 8 && ng == 16) return pick<4, 16, 8>(mode, smallest, a);
    if (w == 16 && ng == 12) return pick<4, 12, 16>(mode, smallest, a);
    if (w == 16 && ng == 16) return pick<4, 16, 16>(mode, smallest, a);
    return hipErrorInvalidValue;
  }
  return hipErrorInvalidValue;
}

}  // namespace rtopk

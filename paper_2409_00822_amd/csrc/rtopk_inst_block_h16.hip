// Instantiations: one workgroup of W wavefronts per row, for rows wider than 8192 columns and few narrower ones -- rows stored as half or bfloat16.
#include "rtopk_block_kernel.hpp"

namespace rtopk {

// 128-bit loads bring 8 values; 6 or 8 loads per lane (W = 4, 8 or 16); few rows with 2 or 4.
template <int G, int NG, int W, int DT>
static hipError_t pick(int mode, const LaunchArgs& a) {
  if (mode == kExact) return launch_block<G, NG, W, kExact, false, DT>(a);
  if (mode == kEarly) return launch_block<G, NG, W, kEarly, false, DT>(a);
  return hipErrorInvalidValue;
}

template <int DT>
static hipError_t pick_shape(int g, int ng, int w, int mode, const LaunchArgs& a) {
  if (g == 8) {
    if (w == 4 && ng == 2) return pick<8, 2, 4, DT>(mode, a);
    if (w == 4 && ng == 4) return pick<8, 4, 4, DT>(mode, a);
    if (w == 8 && ng == 2) return pick<8, 2, 8, DT>(mode, a);
    if (w == 8 && ng == 4) return pick<8, 4, 8, DT>(mode, a);
    if (w == 4 && ng == 6) return pick<8, 6, 4, DT>(mode, a);
    if (w == 4 && ng == 8) return pick<8, 8, 4, DT>(mode, a);
    if (w == 8 && ng == 6) return pick<8, 6, 8, DT>(mode, a);
    if (w == 8 && ng == 8) return pick<8, 8, 8, DT>(mode, a);
    if (w == 16 && ng == 6) return pick<8, 6, 16, DT>(mode, a);
    if (w == 16 && ng == 8) return pick<8, 8, 16, DT>(mode, a);
    return hipErrorInvalidValue;
  }
  return hipErrorInvalidValue;
}

hipError_t launch_block_h16(int dtype, int g, int ng, int w, int mode, const LaunchArgs& a) {
  if (dtype == kF16) return pick_shape<kF16>(g, ng, w, mode, a);
  if (dtype == kBF16) return pick_shape<kBF16>(g, ng, w, mode, a);
  return hipErrorInvalidValue;
}

}  // namespace rtopk

// Instantiations: dense-output form of the selection (chosen values in place, zero elsewhere), fp32.
#include "rtopk_kernel.hpp"

namespace rtopk {

template <int G, int NG, int R, bool FULL>
static hipError_t pick_mode(int mode, const LaunchArgs& a) {
  if (mode == kExact) return launch_dense<G, NG, R, FULL, kExact>(a);
  if (mode == kEarly) return launch_dense<G, NG, R, FULL, kEarly>(a);
  return hipErrorInvalidValue;
}

template <int G, int NG, int R>
static hipError_t pick_rows(bool full, int mode, const LaunchArgs& a) {
  if constexpr (G != 0) {
    if (full) return pick_mode<G, NG, R, true>(mode, a);
  }
  return pick_mode<G, NG, R, false>(mode, a);
}

template <int G, int NG>
static hipError_t pick(bool full, int mode, const LaunchArgs& a) {
  return by_rows_dense<Layout<G, NG>::E>(a.N, [&](auto r) { return pick_rows<G, NG, decltype(r)::value>(full, mode, a); });
}

hipError_t launch_dense_any(int g, int ng, bool full, int mode, const LaunchArgs& a) {
  if (g == 4) {
    switch (ng) {
#define X(n) case n: return pick<4, n>(full, mode, a);
      RTOPK_NG_LIST_G4(X)
#undef X
      default: return hipErrorInvalidValue;
    }
  }
#define X(G, NG) if (g == G && ng == NG) return pick<G, NG>(full, mode, a);
  RTOPK_LAYOUT_LIST_SMALL(X)
#undef X
  return hipErrorInvalidValue;
}

}  // namespace rtopk

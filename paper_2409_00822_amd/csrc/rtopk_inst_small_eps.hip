// Instantiations: fp32 rows of up to 448 columns whose lanes hold one, two, three, five, six or seven values, Algorithm 1 with a relative precision epsilon'.
#include "rtopk_kernel.hpp"

namespace rtopk {

template <int G, int NG, int R>
static hipError_t pick_rows(bool full, const LaunchArgs& a) {
  if constexpr (G != 0) {
    if (full) return launch<G, NG, R, true, kEps, int32_t>(a);
  }
  return launch<G, NG, R, false, kEps, int32_t>(a);
}

template <int G, int NG>
static hipError_t pick(bool full, const LaunchArgs& a) {
  constexpr int E = Layout<G, NG>::E, R = most_rows(E, kPairsEps);
  return by_rows<E, R, kPairsEps>(a.N, [&](auto r) { return pick_rows<G, NG, decltype(r)::value>(full, a); },
                               few_rows_of<E, kPairsEps>(a));
}

hipError_t launch_small_eps(int g, int ng, bool full, const LaunchArgs& a) {
#define X(G, NG) if (g == G && ng == NG) return pick<G, NG>(full, a);
  RTOPK_LAYOUT_LIST_SMALL(X)
#undef X
  return hipErrorInvalidValue;
}

}  // namespace rtopk

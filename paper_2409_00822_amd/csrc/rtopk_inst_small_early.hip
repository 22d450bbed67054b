// Instantiations: fp32 rows of up to 448 columns whose lanes hold one, two, three, five, six or seven values, early mode.
#include "rtopk_kernel.hpp"

namespace rtopk {

// R rows per wavefront; the column type and the k-smallest variant are picked here.
template <int G, int NG, int R, bool FULL>
static hipError_t pick_variant(bool u8, const LaunchArgs& a) {
  if constexpr (Layout<G, NG>::E <= 4) {
    if (u8 && !a.smallest) return launch<G, NG, R, FULL, kEarly, uint8_t>(a);
  }
  if (u8) return hipErrorInvalidValue;
  return a.smallest ? launch<G, NG, R, FULL, kEarly, int32_t, true>(a) : launch<G, NG, R, FULL, kEarly, int32_t>(a);
}

template <int G, int NG, int R>
static hipError_t pick_rows(bool full, bool u8, const LaunchArgs& a) {
  if constexpr (G != 0) {
    if (full) return pick_variant<G, NG, R, true>(u8, a);
  }
  return pick_variant<G, NG, R, false>(u8, a);
}

template <int G, int NG>
static hipError_t pick(bool full, bool u8, const LaunchArgs& a) {
  constexpr int E = Layout<G, NG>::E, R = most_rows(E, kPairs);
  auto rows = [&](auto r) { return pick_rows<G, NG, decltype(r)::value>(full, u8, a); };
  if constexpr (E <= 3) {
    if (u8) return by_rows<E, R, kBytes>(a.N, rows, few_rows_early<E, kBytes>(full, a));
  }
  return by_rows<E, R, kPairs>(a.N, rows, few_rows_early<E, kPairs>(full, a));
}

hipError_t launch_small_early(int g, int ng, bool full, bool u8, const LaunchArgs& a) {
#define X(G, NG) if (g == G && ng == NG) return pick<G, NG>(full, u8, a);
  RTOPK_LAYOUT_LIST_SMALL(X)
#undef X
  return hipErrorInvalidValue;
}

}  // namespace rtopk

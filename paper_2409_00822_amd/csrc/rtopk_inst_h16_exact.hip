// Instantiations: rows stored as IEEE half or bfloat16, exact mode, int32 columns.
#include "rtopk_kernel.hpp"

namespace rtopk {

template <int DT, int G, int NG, int R>
static hipError_t pick_rows(bool full, const LaunchArgs& a) {
  if constexpr (G != 0) {
    if (full) return launch<G, NG, R, true, kExact, int32_t, false, DT>(a);
  }
  return launch<G, NG, R, false, kExact, int32_t, false, DT>(a);
}

template <int DT, int G, int NG>
static hipError_t pick(bool full, const LaunchArgs& a) {
  constexpr int E = Layout<G, NG>::E, R = most_rows(E, kPairs, true);
  if constexpr (E == 16) {
    if (one_row_lists(kExact, true, a)) return pick_rows<DT, G, NG, 1>(full, a);
  }
  return by_rows<E, R, kPairs>(a.N, [&](auto r) { return pick_rows<DT, G, NG, decltype(r)::value>(full, a); },
                               few_rows_of<E, kPairs, true>(a));
}

template <int DT>
static hipError_t pick_shape(int g, int ng, bool full, const LaunchArgs& a) {
  if (g == 8) {
    switch (ng) {
#define X(n) case n: return pick<DT, 8, n>(full, a);
      RTOPK_NG_LIST_H8(X)
#undef X
      default: return hipErrorInvalidValue;
    }
  }
  if (g == 4 && ng == 1) return pick<DT, 4, 1>(full, a);
#define X(G, NG) if (g == G && ng == NG) return pick<DT, G, NG>(full, a);
  RTOPK_LAYOUT_LIST_SMALL(X)
#undef X
  return hipErrorInvalidValue;
}

hipError_t launch_h16_exact(int dtype, int g, int ng, bool full, const LaunchArgs& a) {
  if (dtype == kF16) return pick_shape<kF16>(g, ng, full, a);
  if (dtype == kBF16) return pick_shape<kBF16>(g, ng, full, a);
  return hipErrorInvalidValue;
}

}  // namespace rtopk

// Instantiations: 128-bit-load path (G = 4), Algorithm 1 with a relative precision epsilon'.
#include "rtopk_kernel.hpp"

namespace rtopk {

template <int NG>
static hipError_t pick(bool full, const LaunchArgs& a) {
  constexpr int R = most_rows(4 * NG, kPairsEps);
  return by_rows<4 * NG, R, kPairsEps>(a.N, [&](auto r) {
    constexpr int rows = decltype(r)::value;
    return full ? launch<4, NG, rows, true, kEps, int32_t>(a) : launch<4, NG, rows, false, kEps, int32_t>(a);
  }, few_rows_of<4 * NG, kPairsEps>(a));
}

hipError_t launch_g4_eps(int ng, bool full, const LaunchArgs& a) {
  switch (ng) {
#define X(n) case n: return pick<n>(full, a);
    RTOPK_NG_LIST_G4(X)
#undef X
    default: return hipErrorInvalidValue;
  }
}

}  // namespace rtopk

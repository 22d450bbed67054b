// Instantiations: 128-bit-load path (G = 4), exact mode.
#include "rtopk_kernel.hpp"

namespace rtopk {

// R rows per wavefront; the column type and the k-smallest variant are picked here.
template <int NG, int R>
static hipError_t pick_rows(bool full, bool u8, const LaunchArgs& a) {
  if constexpr (NG == 1) {
    if (u8 && !a.smallest) return full ? launch<4, NG, R, true, kExact, uint8_t>(a) : launch<4, NG, R, false, kExact, uint8_t>(a);
  }
  if (a.smallest) {
    if (u8) return hipErrorInvalidValue;
    return full ? launch<4, NG, R, true, kExact, int32_t, true>(a) : launch<4, NG, R, false, kExact, int32_t, true>(a);
  }
  return full ? launch<4, NG, R, true, kExact, int32_t>(a) : launch<4, NG, R, false, kExact, int32_t>(a);
}

template <int NG>
static hipError_t pick(bool full, bool u8, const LaunchArgs& a) {
  constexpr int R = rows_per_wave(4 * NG);
  if constexpr (NG == 4) {
    if (one_row_lists(kExact, false, a)) return pick_rows<NG, 1>(full, u8, a);
  }
  auto rows = [&](auto r) { return pick_rows<NG, decltype(r)::value>(full, u8, a); };
  if constexpr (NG == 1) {
    if (u8) return full ? by_rows<4, kRowsPerWaveFp32M256, kBytes>(a.N, rows) : by_rows<4, R, kBytes>(a.N, rows);
    return by_rows<4, R, kPairs>(a.N, rows, few_rows_of<4, kPairs>(a));
  }
  return by_rows<4 * NG, R, kPairs>(a.N, rows);
}

hipError_t launch_g4_exact(int ng, bool full, bool u8, const LaunchArgs& a) {
  switch (ng) {
#define X(n) case n: return pick<n>(full, u8, a);
    RTOPK_NG_LIST_G4(X)
#undef X
    default: return hipErrorInvalidValue;
  }
}

}  // namespace rtopk

// Instantiations: fp32 rows of more than 32768 columns spread over several workgroups, with scratch memory.
#include "rtopk_split_kernel.hpp"

namespace rtopk {

static Split split_for(int64_t N, int M, int k, int mode, int max_iter) {
  const Split s = split_of(N, M, k, mode, max_iter);
  return s.segments > 0 ? s : split_big_of(N, M, k, mode, max_iter);
}

int64_t split_scratch_bytes(int64_t N, int M, int k, int mode, int max_iter) {
  const Split s = split_for(N, M, k, mode, max_iter);
  return s.segments > 0 ? s.bytes() : 0;
}

hipError_t launch_split_any(int mode, bool smallest, void* scratch, const LaunchArgs& a) {
  const Split s = split_for(a.N, a.M, a.k, mode, a.max_iter);
  if (s.segments == 0) return hipErrorInvalidValue;
  if (smallest) {
    if (mode == kExact) return launch_split<kExact, true>(s, scratch, a);
    if (mode == kEarly) return launch_split<kEarly, true>(s, scratch, a);
    return hipErrorInvalidValue;
  }
  if (mode == kExact) return launch_split<kExact, false>(s, scratch, a);
  if (mode == kEarly) return launch_split<kEarly, false>(s, scratch, a);
  if (mode == kEps) return launch_split<kEps, false>(s, scratch, a);
  return hipErrorInvalidValue;
}

}  // namespace rtopk

// Instantiations: fp32 rows of more than 32768 columns spread over several workgroups, with scratch memory.
#include "rtopk_split_kernel.hpp"

namespace rtopk {

hipError_t launch_split_any(const Split& s, int mode, bool smallest, void* scratch, const LaunchArgs& a) {
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

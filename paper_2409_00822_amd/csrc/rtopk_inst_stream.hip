// Instantiations: rows wider than 65536 columns, streamed (fp32 rows, int32 columns).
#include "rtopk_stream_kernel.hpp"

namespace rtopk {

hipError_t launch_stream_any(int mode, bool smallest, const LaunchArgs& a) {
  if (smallest) {
    if (mode == kExact) return launch_stream<kExact, true>(a);
    if (mode == kEarly) return launch_stream<kEarly, true>(a);
    return hipErrorInvalidValue;
  }
  if (mode == kExact) return launch_stream<kExact, false>(a);
  if (mode == kEarly) return launch_stream<kEarly, false>(a);
  if (mode == kEps) return launch_stream<kEps, false>(a);
  return hipErrorInvalidValue;
}

}  // namespace rtopk

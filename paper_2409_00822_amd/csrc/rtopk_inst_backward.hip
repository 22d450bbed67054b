// Instantiations: backward edge of the MaxK non-linearity (scatter and gather forms, int32 and uint8 columns).
#include "rtopk_backward.hpp"

namespace rtopk {

hipError_t launch_maxk_backward(const float* grad_vals, const void* idx, bool u8, int64_t N, int M, int k, float* grad_in,
                                hipStream_t stream) {
  return u8 ? launch_scatter(grad_vals, static_cast<const uint8_t*>(idx), N, M, k, grad_in, stream)
            : launch_scatter(grad_vals, static_cast<const int32_t*>(idx), N, M, k, grad_in, stream);
}

hipError_t launch_maxk_backward_gather(const float* grad_out, const void* idx, bool u8, int64_t N, int M, int k,
                                       float* grad_vals, hipStream_t stream) {
  return u8 ? launch_gather(grad_out, static_cast<const uint8_t*>(idx), N, M, k, grad_vals, stream)
            : launch_gather(grad_out, static_cast<const int32_t*>(idx), N, M, k, grad_vals, stream);
}

}  // namespace rtopk

// Host-side dispatch table between the C ABI (rtopk_api.hip) and the kernel instantiations, which
// are spread over several translation units so that they compile in parallel.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rtopk_shape.hpp"

namespace rtopk {

struct LaunchArgs {
  const void* in;
  int64_t N;
  int M, k, max_iter;
  float eps_rel;       // kEps only
  int32_t* out_iters;  // kEps only, may be null
  bool smallest;       // select the k smallest instead of the k largest (kEarly / kExact, int32 columns)
  void* out_vals;
  void* out_idx;
  int vec_store;  // both outputs are aligned to four of their elements: 1 where k % 4 == 0, 2 otherwise; else 0
  hipStream_t stream;
};

// fp32 rows of up to 8192 columns, one wavefront per row.  g = columns per group, ng = groups per lane
// (M <= 64*g*ng), as kernel_layout() returns them; full = (M == 64*g*ng): no column-validity tests in the kernel.
hipError_t launch_g4_exact(int ng, bool full, bool u8, const LaunchArgs& a);
hipError_t launch_g4_early(int ng, bool full, bool u8, const LaunchArgs& a);
hipError_t launch_g4_eps(int ng, bool full, const LaunchArgs& a);  // int32 columns only
// g = 1 or 2 with ng = 1, or g = 0: ng values per lane in groups of mixed width.
hipError_t launch_small_exact(int g, int ng, bool full, bool u8, const LaunchArgs& a);
hipError_t launch_small_early(int g, int ng, bool full, bool u8, const LaunchArgs& a);
hipError_t launch_small_eps(int g, int ng, bool full, const LaunchArgs& a);  // int32 columns only
// The same for rows stored in 16 bits (dtype kF16 or kBF16; kEarly / kExact, int32 columns).
hipError_t launch_h16_exact(int dtype, int g, int ng, bool full, const LaunchArgs& a);
hipError_t launch_h16_early(int dtype, int g, int ng, bool full, const LaunchArgs& a);
// Rows wider than 8192 columns: one workgroup of w wavefronts per row (int32 columns).  g = elements per
// load (4 for fp32 / 8 for 16-bit rows), ng = loads per lane, M <= 64*w*g*ng.
hipError_t launch_block_plain(int g, int ng, int w, int mode, const LaunchArgs& a);                   // fp32, kEarly / kExact
hipError_t launch_block_variant(int g, int ng, int w, int mode, bool smallest, const LaunchArgs& a);  // fp32: kEps, or the k smallest
hipError_t launch_block_dense(int g, int ng, int w, int mode, const LaunchArgs& a);                   // fp32 dense output
hipError_t launch_block_h16(int dtype, int g, int ng, int w, int mode, const LaunchArgs& a);          // half / bfloat16 rows
// Rows wider than 65536 columns (fp32, int32 columns, every mode, the k largest or smallest): one
// workgroup per row, the row streamed.
hipError_t launch_stream_any(int mode, bool smallest, const LaunchArgs& a);
// fp32 rows of more than 32768 columns over several workgroups each, in two launches; s: split_for, not empty.
hipError_t launch_split_any(const Split& s, int mode, bool smallest, void* scratch, const LaunchArgs& a);
// Dense-output form (fp32; a.out_vals is the [N][M] output, a.out_idx unused).  g, ng, full as above;
// mode kEarly or kExact.
hipError_t launch_dense_any(int g, int ng, bool full, int mode, const LaunchArgs& a);

// Backward edge of the MaxK non-linearity (rtopk_backward.hpp).  idx is int32_t[N][k] or, with u8,
// uint8_t[N][k].
hipError_t launch_maxk_backward(const float* grad_vals, const void* idx, bool u8, int64_t N, int M, int k, float* grad_in,
                                hipStream_t stream);
hipError_t launch_maxk_backward_gather(const float* grad_out, const void* idx, bool u8, int64_t N, int M, int k,
                                       float* grad_vals, hipStream_t stream);

}  // namespace rtopk

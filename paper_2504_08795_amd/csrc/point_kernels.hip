// Depthwise convolution and max pooling for windows whose size is known at compile time (layer_bodies.h).
#include <hip/hip_runtime.h>

#include "layer_bodies.h"
#include "device_common.h"
#include "kernels.h"

namespace daris {

template <bool BF16, int K>
__global__ __launch_bounds__(256) void dwconv_window_kernel(const DwWindowArgs) {
  const DwWindowArgs p = args_at<DwWindowArgs>((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr());
  dwconv_point<BF16, K>(p.a, point_of<BF16>(p.a, p.at, (int)blockIdx.x, (int)threadIdx.x));
  puts_done();
}

template <bool BF16, int K>
__global__ __launch_bounds__(256) void maxpool_window_kernel(const PoolWindowArgs) {
  const PoolWindowArgs p = args_at<PoolWindowArgs>((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr());
  maxpool_point<BF16, K>(p.a, point_of<BF16>(p.a, p.at, (int)blockIdx.x, (int)threadIdx.x));
  puts_done();
}

#define DARIS_INST_POINT(B)                                              \
  template __global__ void dwconv_window_kernel<B, 3>(const DwWindowArgs);    \
  template __global__ void maxpool_window_kernel<B, 2>(const PoolWindowArgs); \
  template __global__ void maxpool_window_kernel<B, 3>(const PoolWindowArgs);
DARIS_INST_POINT(false)
DARIS_INST_POINT(true)
#undef DARIS_INST_POINT

}  // namespace daris

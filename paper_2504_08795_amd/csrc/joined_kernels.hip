// Kernels that compute layers which follow one another in one launch (layer_bodies.h).
#include <hip/hip_runtime.h>

#include "layer_bodies.h"
#include "device_common.h"
#include "kernels.h"

namespace daris {

// The first convolution of a network and the max pooling behind it.
template <bool BF16>
__global__ __launch_bounds__(128 * (kImagePoolRows + 1)) void conv_image_pool_kernel(const ImageConvArgs) {
  ImageConvArgs p = grab<ImageConvArgs>((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr());
  args_in_memory(p);
  __shared__ __align__(16) float lds[conv_image_lds<BF16, true>()];
  conv_image_body<BF16, 2, true>(p, (int)blockIdx.x, lds);
  puts_done();
}

template __global__ void conv_image_pool_kernel<false>(const ImageConvArgs);
template __global__ void conv_image_pool_kernel<true>(const ImageConvArgs);

// A 1x1 convolution and the depthwise convolution behind it.
template <bool BF16, int NCH>
__global__ __launch_bounds__(512) void conv_expand_dw_kernel(const ExpandDwArgs) {
  ExpandDwArgs p = grab<ExpandDwArgs>((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr());
  p.dw_w = in_memory(p.dw_w);
  p.dw_bias = in_memory(p.dw_bias);
  args_in_memory(p);
  __shared__ __align__(16) float lds[kExpandPixels * kExpandRow + 160];
  conv_expand_dw_body<BF16, NCH>(p, (int)blockIdx.x, lds);
  puts_done();
}

#define DARIS_INST_EXPAND(B)                                            \
  template __global__ void conv_expand_dw_kernel<B, 1>(const ExpandDwArgs); \
  template __global__ void conv_expand_dw_kernel<B, 2>(const ExpandDwArgs); \
  template __global__ void conv_expand_dw_kernel<B, 3>(const ExpandDwArgs); \
  template __global__ void conv_expand_dw_kernel<B, 4>(const ExpandDwArgs); \
  template __global__ void conv_expand_dw_kernel<B, 5>(const ExpandDwArgs);
DARIS_INST_EXPAND(false)
DARIS_INST_EXPAND(true)
#undef DARIS_INST_EXPAND

}  // namespace daris

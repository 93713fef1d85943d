// The first convolution of a network, reading the caller's input (conv_image_body in layer_bodies.h).
#include <hip/hip_runtime.h>

#include "layer_bodies.h"
#include "device_common.h"
#include "kernels.h"

namespace daris {

template <bool BF16, int WN>
__global__ __launch_bounds__(256) void conv_image_kernel(const ImageConvArgs) {
  ImageConvArgs p = grab<ImageConvArgs>((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr());
  args_in_memory(p);
  __shared__ __align__(16) float lds[conv_image_lds<BF16, false>()];
  conv_image_body<BF16, WN, false>(p, (int)blockIdx.x, lds);
  puts_done();
}

template __global__ void conv_image_kernel<false, 1>(const ImageConvArgs);
template __global__ void conv_image_kernel<false, 2>(const ImageConvArgs);
template __global__ void conv_image_kernel<true, 1>(const ImageConvArgs);
template __global__ void conv_image_kernel<true, 2>(const ImageConvArgs);

}  // namespace daris

// Implicit-GEMM convolution of large fp32 layers on gfx950: 64 pixels x 64 channels per wave (block_body.h).
#include <hip/hip_runtime.h>

#include "block_body.h"
#include "device_common.h"
#include "kernels.h"

namespace daris {

template <int NW, bool TAPS>
__global__ __launch_bounds__(NW * 64) void conv_block_kernel(const ConvArgs) {
  const ConvArgs p = conv_args_at((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr());
  __shared__ __align__(16) float red[conv_block_lds<NW, TAPS>()];
  conv_block_body<NW, TAPS, false>(p, red);
  puts_done();
}

template __global__ void conv_block_kernel<2, false>(const ConvArgs);
template __global__ void conv_block_kernel<4, false>(const ConvArgs);
template __global__ void conv_block_kernel<8, false>(const ConvArgs);
template __global__ void conv_block_kernel<2, true>(const ConvArgs);
template __global__ void conv_block_kernel<4, true>(const ConvArgs);
template __global__ void conv_block_kernel<8, true>(const ConvArgs);

}  // namespace daris

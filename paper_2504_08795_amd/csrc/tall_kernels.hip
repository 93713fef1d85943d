// Tiles of two blocks of pixels and one of channels with three taps per fetch (conv_taps_body in layer_bodies.h).
#include <hip/hip_runtime.h>

#include "layer_bodies.h"
#include "device_common.h"
#include "kernels.h"

namespace daris {

template <bool BF16>
__global__ __launch_bounds__(512, 4) void conv_taps16_tall_kernel(const ConvArgs) {
  const ConvArgs p = conv_args_at((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr());
  __shared__ __align__(16) float red[conv_taps_lds<BF16, 16, 1, 8, 2>()];
  int mt, g;
  if (!conv_tile_of(p, (int)blockIdx.x, &mt, &g)) return;
  conv_taps_body<BF16, 16, 1, 8, false, 2>(p, mt, g, red);
  puts_done();
}

// for the plans of conv_taps16_kernel<., 2, 8>
template __global__ void conv_taps16_tall_kernel<false>(const ConvArgs);
template __global__ void conv_taps16_tall_kernel<true>(const ConvArgs);

}  // namespace daris

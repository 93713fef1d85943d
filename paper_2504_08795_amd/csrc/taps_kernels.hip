// Convolutions whose waves fetch rows once for three taps of a 3 x 3 window (conv_taps_body in layer_bodies.h).
#include <hip/hip_runtime.h>

#include "layer_bodies.h"
#include "device_common.h"
#include "kernels.h"

namespace daris {

template <bool BF16, int TN, int NW>
__global__ __launch_bounds__(NW * 64) void conv_taps_kernel(const ConvArgs) {
  const ConvArgs p = conv_args_at((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr());
  __shared__ __align__(16) float red[conv_taps_lds<BF16, 32, TN, NW>()];
  int mt, g;
  if (!conv_tile_of(p, (int)blockIdx.x, &mt, &g)) return;
  conv_taps_body<BF16, 32, TN, NW>(p, mt, g, red);
  puts_done();
}

template <bool BF16, int TB, int NW>
__global__ __launch_bounds__(NW * 64, NW == 8 ? 4 : 1) void conv_taps16_kernel(const ConvArgs) {
  const ConvArgs p = conv_args_at((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr());
  __shared__ __align__(16) float red[conv_taps_lds<BF16, 16, TB, NW>()];
  int mt, g;
  if (!conv_tile_of(p, (int)blockIdx.x, &mt, &g)) return;
  conv_taps_body<BF16, 16, TB, NW>(p, mt, g, red);
  puts_done();
}

// Tensors of 2 GiB and more, as conv_large_kernel.
template <bool BF16, int TN>
__global__ __launch_bounds__(128) void conv_taps_large_kernel(const ConvArgs) {
  const ConvArgs p = conv_args_at((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr());
  __shared__ __align__(16) float red[conv_taps_lds<BF16, 32, TN, 2>()];
  int mt, g;
  if (!conv_tile_of(p, (int)blockIdx.x, &mt, &g)) return;
  conv_taps_body<BF16, 32, TN, 2, true>(p, mt, g, red);
  puts_done();
}

// The tiles and numbers of waves that the planner arrives at (taps_kernel in launch.cpp).  For 32 pixels these are two, four or eight in fp32 (not
// four with 64 channels: what would have them has too few groups of taps, or 64 x 64 tiles), two or four in bf16; for 16 pixels
// eight in fp32, four or eight in bf16.
#define DARIS_INST_TAPS(B, T, W) template __global__ void conv_taps_kernel<B, T, W>(const ConvArgs);
#define DARIS_INST_TAPS16(B, W) \
  template __global__ void conv_taps16_kernel<B, 1, W>(const ConvArgs); \
  template __global__ void conv_taps16_kernel<B, 2, W>(const ConvArgs);
DARIS_INST_TAPS(false, 1, 2) DARIS_INST_TAPS(false, 1, 4) DARIS_INST_TAPS(false, 1, 8) DARIS_INST_TAPS(false, 2, 2) DARIS_INST_TAPS(false, 2, 8)
DARIS_INST_TAPS(true, 1, 2) DARIS_INST_TAPS(true, 1, 4) DARIS_INST_TAPS(true, 2, 2) DARIS_INST_TAPS(true, 2, 4)
DARIS_INST_TAPS16(false, 8)
DARIS_INST_TAPS16(true, 4) DARIS_INST_TAPS16(true, 8)
template __global__ void conv_taps_large_kernel<false, 1>(const ConvArgs);
template __global__ void conv_taps_large_kernel<false, 2>(const ConvArgs);
template __global__ void conv_taps_large_kernel<true, 1>(const ConvArgs);
template __global__ void conv_taps_large_kernel<true, 2>(const ConvArgs);
#undef DARIS_INST_TAPS16
#undef DARIS_INST_TAPS

}  // namespace daris

// 1x1 convolutions over whole rows (conv_rows_body with POINT), alone and two in a launch.
#include <hip/hip_runtime.h>

#include "layer_bodies.h"
#include "device_common.h"
#include "kernels.h"

namespace daris {

template <bool BF16, int R, int TN, int NW>
constexpr int point_lds() {  // floats of LDS
  return R == 16 ? conv_rows_lds<16, TN, NW>() : conv_wave_lds<BF16, TN, NW, 3>();
}
// (three waves a SIMD as conv_wave_kernel has them)
template <bool BF16, int R, int TN, int NW>
__global__ __launch_bounds__(NW * 64, BF16 && R == 32 && TN == 2 ? 3 : 1) void conv_point_kernel(const ConvArgs) {
  const ConvArgs p = conv_args_at((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr());
  __shared__ __align__(16) float red[point_lds<BF16, R, TN, NW>()];
  int mt, g;
  if (!conv_tile_of(p, (int)blockIdx.x, &mt, &g)) return;
  conv_rows_body<BF16, R, TN, NW, false, true>(p, mt, g, red);
  puts_done();
}

// As conv_wave_pair_kernel: workgroups [0, n0) work on the first problem.
template <bool BF16, int R, int TN, int NW>
__global__ __launch_bounds__(NW * 64, BF16 && R == 32 && TN == 2 ? 3 : 1) void conv_point_pair_kernel(const ConvArgs, const ConvArgs, const int n0) {
  __shared__ __align__(16) float red[point_lds<BF16, R, TN, NW>()];
  const bool second = (int)blockIdx.x >= n0;
  const ConvArgs p = conv_args_at((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr() + (second ? sizeof(ConvArgs) : 0));
  int mt, g;
  if (!conv_tile_of(p, (int)blockIdx.x - (second ? n0 : 0), &mt, &g)) return;
  conv_rows_body<BF16, R, TN, NW, false, true>(p, mt, g, red);
  puts_done();
}

#define DARIS_INST_POINT(B, R, T, W)                                \
  template __global__ void conv_point_kernel<B, R, T, W>(const ConvArgs); \
  template __global__ void conv_point_pair_kernel<B, R, T, W>(const ConvArgs, const ConvArgs, const int);
#define DARIS_INST_POINT_W(B, R, T) DARIS_INST_POINT(B, R, T, 2) DARIS_INST_POINT(B, R, T, 4) DARIS_INST_POINT(B, R, T, 8)
#define DARIS_INST_POINT_T(B, R) DARIS_INST_POINT_W(B, R, 1) DARIS_INST_POINT_W(B, R, 2)
DARIS_INST_POINT_T(false, 32)
DARIS_INST_POINT(true, 32, 1, 2) DARIS_INST_POINT(true, 32, 1, 4) DARIS_INST_POINT(true, 32, 2, 2) DARIS_INST_POINT(true, 32, 2, 4)  // (no bf16 plan of 32-pixel tiles has eight waves)
DARIS_INST_POINT_T(false, 16)
DARIS_INST_POINT_T(true, 16)
#undef DARIS_INST_POINT_T
#undef DARIS_INST_POINT_W
#undef DARIS_INST_POINT

}  // namespace daris

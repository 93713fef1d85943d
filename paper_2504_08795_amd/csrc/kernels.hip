// HIP kernels of the DNN stages for gfx950 (CDNA4): implicit-GEMM convolution on MFMA with register-fed wave tiles
// and a fused bias / residual / activation epilogue, split-K reduction, depthwise convolution, pooling, FC
// (batch-1 GEMV), and the NCHW<->NHWC boundary conversions.  A DNN is, for the scheduler of the paper
// (Sec. I, Sec. III-B1), a sequence of such kernels cut into stages.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "layer_bodies.h"
#include "device_common.h"
#include "kernels.h"

namespace daris {

// Sums the split-K partials in split order and applies the fused epilogue.  One thread per 4 output channels.
// Partials travel four at a time, one trip to memory per four slices.
template <bool BF16>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ ws, const float* __restrict__ bias,
                                                            const void* res, void* y, int M, int N, int splitk, int act) {
  const uint32_t idx = blockIdx.x * 256u + threadIdx.x, n4 = (uint32_t)N >> 2;
  const size_t o = (size_t)idx * 4;
  const uint32_t row = idx / n4;
  if (row >= (uint32_t)M) return;
  const int n = (int)(idx - row * n4) * 4;
  const float4 b = *(const float4*)(bias + n);
  const size_t slice = (size_t)M * N;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int z = 0; z < splitk; z += 4) {
    float4 t[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) t[u] = *(const float4*)(ws + (size_t)min(z + u, splitk - 1) * slice + o);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (z + u < splitk) {  // (slice 0 as it is: 0 + -0 would lose the sign)
        const bool first = z + u == 0;
        s.x = first ? t[u].x : s.x + t[u].x; s.y = first ? t[u].y : s.y + t[u].y;
        s.z = first ? t[u].z : s.z + t[u].z; s.w = first ? t[u].w : s.w + t[u].w;
      }
  }
  float v[4] = {s.x + b.x, s.y + b.y, s.z + b.z, s.w + b.w};
  if (res) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] += load_elem<BF16>(res, o + i);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = apply_act(v[i], act);
  if (BF16) {
    uint2 out;
    out.x = pack_bf16_rne(v[0], v[1]);
    out.y = pack_bf16_rne(v[2], v[3]);
    put((uint16_t*)y + o, out);
  } else {
    put((float*)y + o, make_float4(v[0], v[1], v[2], v[3]));
  }
  puts_done();
}

// ---- wave-tile implicit GEMM (layer_bodies.h), one tile per workgroup ------------------------------------------------------
// Waves that a SIMD is to have the registers for: three of the 32 x 64 tiles over whole rows in bf16, which stay within 168 each so (one more with two waves a
// workgroup otherwise; see rows_pipeline).
template <bool BF16, int TN, int NW, int MODE>
constexpr int waves_per_simd() {
  return BF16 && TN == 2 && NW < 8 && MODE == 3 ? 3 : 1;
}
template <bool BF16, int TN, int NW, int MODE>
__global__ __launch_bounds__(NW * 64, (waves_per_simd<BF16, TN, NW, MODE>())) void conv_wave_kernel(const ConvArgs) {
  const ConvArgs p = conv_args_at((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr());
  __shared__ __align__(16) float red[conv_wave_lds<BF16, TN, NW, MODE>()];
  int mt, g;
  if (!conv_tile_of(p, (int)blockIdx.x, &mt, &g)) return;
  if constexpr (MODE == 3) conv_rows_body<BF16, 32, TN, NW>(p, mt, g, red);
  else conv_wave_body<BF16, TN, NW, MODE, 2>(p, mt, g, red, DwFusedArgs());
  puts_done();
}

// Whole rows of tensors of 2 GiB and more; their grids are large, so that their plans have two waves a workgroup.
template <bool BF16, int TN>
__global__ __launch_bounds__(128, (waves_per_simd<BF16, TN, 2, 3>())) void conv_large_kernel(const ConvArgs) {
  const ConvArgs p = conv_args_at((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr());
  __shared__ __align__(16) float red[conv_wave_lds<BF16, TN, 2, 3>()];
  int mt, g;
  if (!conv_tile_of(p, (int)blockIdx.x, &mt, &g)) return;
  conv_rows_body<BF16, 32, TN, 2, true>(p, mt, g, red);
  puts_done();
}

// A 1x1 convolution with the 3x3 depthwise convolution in front of it computed on the fly (gather mode 4): one launch for
// the second and third layer of an inverted residual block, and the depthwise output never touches memory.
template <bool BF16, int TN, int NW>
__global__ __launch_bounds__(NW * 64) void conv_wave_dw_kernel(const ConvArgs, const DwFusedArgs d) {
  const ConvArgs p = conv_args_at((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr());
  __shared__ __align__(16) float red[conv_wave_lds<BF16, TN, NW, 4>()];
  int mt, g;
  if (!conv_tile_of(p, (int)blockIdx.x, &mt, &g)) return;
  conv_wave_body<BF16, TN, NW, 4, 1>(p, mt, g, red, d);
  puts_done();
}
// Two independent convolutions of the same kernel variant in one launch (a residual block's first convolution and
// the 1x1 convolution of its shortcut read the same tensor): workgroups [0, n0) work on p0, the rest on p1.  n0 is
// a multiple of 8, so the workgroup -> XCD relation of each problem is the one its plan assumed.
template <bool BF16, int TN, int NW, int MODE>
__global__ __launch_bounds__(NW * 64, (waves_per_simd<BF16, TN, NW, MODE>())) void conv_wave_pair_kernel(const ConvArgs, const ConvArgs, const int n0) {
  __shared__ __align__(16) float red[conv_wave_lds<BF16, TN, NW, MODE>()];
  const bool second = (int)blockIdx.x >= n0;
  const ConvArgs p = conv_args_at((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr() + (second ? sizeof(ConvArgs) : 0));
  int mt, g;
  if (!conv_tile_of(p, (int)blockIdx.x - (second ? n0 : 0), &mt, &g)) return;
  if constexpr (MODE == 3) conv_rows_body<BF16, 32, TN, NW>(p, mt, g, red);
  else conv_wave_body<BF16, TN, NW, MODE, 2>(p, mt, g, red, DwFusedArgs());
  puts_done();
}

template <bool BF16, int TB, int NW>
__global__ __launch_bounds__(NW * 64) void conv_wave16_kernel(const ConvArgs) {
  const ConvArgs p = conv_args_at((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr());
  __shared__ __align__(16) float red[conv_rows_lds<16, TB, NW>()];
  int mt, g;
  if (!conv_tile_of(p, (int)blockIdx.x, &mt, &g)) return;
  conv_rows_body<BF16, 16, TB, NW>(p, mt, g, red);
  puts_done();
}

// Two independent convolutions on one tensor in one launch, as conv_wave_pair_kernel: workgroups [0, n0) work on p0.
template <bool BF16, int TB, int NW>
__global__ __launch_bounds__(NW * 64) void conv_wave16_pair_kernel(const ConvArgs, const ConvArgs, const int n0) {
  __shared__ __align__(16) float red[conv_rows_lds<16, TB, NW>()];
  const bool second = (int)blockIdx.x >= n0;
  const ConvArgs p = conv_args_at((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr() + (second ? sizeof(ConvArgs) : 0));
  int mt, g;
  if (!conv_tile_of(p, (int)blockIdx.x - (second ? n0 : 0), &mt, &g)) return;
  conv_rows_body<BF16, 16, TB, NW>(p, mt, g, red);
  puts_done();
}

// ---- the memory-bound layers (layer_bodies.h) -----------------------------------------------------------------------------
template <bool BF16>
__global__ __launch_bounds__(256) void dwconv_kernel(const DwArgs a) {
  dwconv_point<BF16, 0>(a, point_of<BF16>(a, blockIdx.x * 256u + threadIdx.x));
  puts_done();
}

template <bool BF16>
__global__ __launch_bounds__(256) void maxpool_kernel(const PoolArgs) {
  const PoolArgs a = args_at<PoolArgs>((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr());
  maxpool_point<BF16, 0>(a, point_of<BF16>(a, blockIdx.x * 256u + threadIdx.x));
  puts_done();
}

template <bool BF16>
__global__ __launch_bounds__(256) void gavgpool_kernel(const PoolArgs) {
  const PoolArgs a = args_at<PoolArgs>((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr());
  __shared__ float part[4][64];
  gavgpool_group<BF16>(a, (int)blockIdx.x, (int)threadIdx.x, part);
  puts_done();
}

template <bool BF16>
__global__ __launch_bounds__(256) void fc_kernel(const FcArgs) {
  const FcArgs a = args_at<FcArgs>((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr());
  fc_row<BF16>(a, (int)(blockIdx.x * 4 + (threadIdx.x >> 6)), (int)(threadIdx.x & 63));
  puts_done();
}

// ---- boundary conversions ------------------------------------------------------------------------------------------------
template <bool BF16>
__global__ __launch_bounds__(256) void ingest_kernel(const float* __restrict__ x, void* y, int C, int Cs, int HW) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (size_t)HW * Cs) return;
  const int c = (int)(idx % Cs);
  const size_t px = idx / Cs;
  put_elem<BF16>(y, idx, c < C ? x[(size_t)c * HW + px] : 0.f);
  puts_done();
}

template <bool BF16>
__global__ __launch_bounds__(256) void egress_kernel(const void* x, float* __restrict__ y, int C, int Cs, int HW) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (size_t)HW * C) return;
  const int c = (int)(idx / HW);
  const size_t px = idx % HW;
  put(y + idx, load_elem<BF16>(x, px * Cs + c));
  puts_done();
}

// ---- CU mask probe: which XCC / CU did each workgroup run on ----------------------------------------------------------------
__global__ __launch_bounds__(64) void cu_probe_kernel(uint32_t* out, int spin) {
  uint32_t xcc, hwid;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_HW_ID)" : "=s"(hwid));
  // bounded busy wait so that the workgroups of one launch spread over every CU the mask allows
  for (int i = 0; i < spin; ++i) __builtin_amdgcn_s_sleep(8);
  if (threadIdx.x == 0) {
    out[2 * blockIdx.x] = xcc;
    out[2 * blockIdx.x + 1] = hwid;
  }
}

// ---- explicit instantiations: the host never references the kernels (they are dispatched by name from the code object) --------
#define DARIS_INST_CONV(B, TN_, NW_)                                                              \
  template __global__ void conv_wave_kernel<B, TN_, NW_, 1>(const ConvArgs);                      \
  template __global__ void conv_wave_kernel<B, TN_, NW_, 2>(const ConvArgs);                      \
  template __global__ void conv_wave_kernel<B, TN_, NW_, 3>(const ConvArgs);                      \
  template __global__ void conv_wave_pair_kernel<B, TN_, NW_, 1>(const ConvArgs, const ConvArgs, const int); \
  template __global__ void conv_wave_pair_kernel<B, TN_, NW_, 3>(const ConvArgs, const ConvArgs, const int);
#define DARIS_INST_CONV_ALIGNED(TN_, NW_) /* gather mode 0: bf16 only */                          \
  template __global__ void conv_wave_kernel<true, TN_, NW_, 0>(const ConvArgs);                   \
  template __global__ void conv_wave_pair_kernel<true, TN_, NW_, 0>(const ConvArgs, const ConvArgs, const int);
#define DARIS_INST_CONV16(B, TB_)                                                                  \
  template __global__ void conv_wave16_kernel<B, TB_, 2>(const ConvArgs);                          \
  template __global__ void conv_wave16_kernel<B, TB_, 4>(const ConvArgs);                          \
  template __global__ void conv_wave16_kernel<B, TB_, 8>(const ConvArgs);                          \
  template __global__ void conv_wave16_pair_kernel<B, TB_, 2>(const ConvArgs, const ConvArgs, const int); \
  template __global__ void conv_wave16_pair_kernel<B, TB_, 4>(const ConvArgs, const ConvArgs, const int); \
  template __global__ void conv_wave16_pair_kernel<B, TB_, 8>(const ConvArgs, const ConvArgs, const int);
#define DARIS_INST_CONVDW(B, TN_, NW_)                                                             \
  template __global__ void conv_wave_dw_kernel<B, TN_, NW_>(const ConvArgs, const DwFusedArgs);
#define DARIS_INST_ALL(B)                                                                          \
  DARIS_INST_CONV(B, 1, 2) DARIS_INST_CONV(B, 1, 4) DARIS_INST_CONV(B, 1, 8)                        \
  DARIS_INST_CONV(B, 2, 2) DARIS_INST_CONV(B, 2, 4) DARIS_INST_CONV(B, 2, 8)                        \
  DARIS_INST_CONV16(B, 1) DARIS_INST_CONV16(B, 2)                                                   \
  template __global__ void splitk_reduce_kernel<B>(const float*, const float*, const void*, void*, int, int, int, int); \
  template __global__ void dwconv_kernel<B>(const DwArgs);                                         \
  template __global__ void maxpool_kernel<B>(const PoolArgs);                                      \
  template __global__ void gavgpool_kernel<B>(const PoolArgs);                                     \
  template __global__ void fc_kernel<B>(const FcArgs);                                             \
  template __global__ void ingest_kernel<B>(const float*, void*, int, int, int);                   \
  template __global__ void egress_kernel<B>(const void*, float*, int, int, int);
DARIS_INST_ALL(false)
DARIS_INST_ALL(true)
DARIS_INST_CONV_ALIGNED(1, 2) DARIS_INST_CONV_ALIGNED(1, 4) DARIS_INST_CONV_ALIGNED(1, 8)
DARIS_INST_CONV_ALIGNED(2, 2) DARIS_INST_CONV_ALIGNED(2, 4) DARIS_INST_CONV_ALIGNED(2, 8)
// Fused depthwise variants.  In fp32 for 32-channel tiles only: with 64 channels they take 249 to 300 registers, and no projection of
// MobileNetV2 with enough pixels has more than 24; bf16 plans never use 8 waves per workgroup, and those variants would need scratch memory, which the dispatch path
// does not provide.
DARIS_INST_CONVDW(false, 1, 2) DARIS_INST_CONVDW(false, 1, 4) DARIS_INST_CONVDW(false, 1, 8)
DARIS_INST_CONVDW(true, 1, 2) DARIS_INST_CONVDW(true, 1, 4) DARIS_INST_CONVDW(true, 2, 2) DARIS_INST_CONVDW(true, 2, 4)
template __global__ void conv_large_kernel<false, 1>(const ConvArgs);
template __global__ void conv_large_kernel<false, 2>(const ConvArgs);
template __global__ void conv_large_kernel<true, 1>(const ConvArgs);
template __global__ void conv_large_kernel<true, 2>(const ConvArgs);
#undef DARIS_INST_CONVDW
#undef DARIS_INST_ALL
#undef DARIS_INST_CONV
#undef DARIS_INST_CONV_ALIGNED
#undef DARIS_INST_CONV16

}  // namespace daris

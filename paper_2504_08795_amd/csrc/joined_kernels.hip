// Kernels that compute layers which follow one another in one launch (layer_bodies.h).
#include <hip/hip_runtime.h>

#include "block_body.h"
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

// A large fp32 convolution with three taps per fetch and the 2 x 2 max pooling behind it.
template <int NW>
__global__ __launch_bounds__(NW * 64) void conv_block_pool_kernel(const ConvArgs) {
  const ConvArgs p = conv_args_at((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr());
  __shared__ __align__(16) float red[conv_block_lds<NW, true>()];
  conv_block_body<NW, true, true>(p, red);
  puts_done();
}
template __global__ void conv_block_pool_kernel<2>(const ConvArgs);
template __global__ void conv_block_pool_kernel<4>(const ConvArgs);
template __global__ void conv_block_pool_kernel<8>(const ConvArgs);

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

// A 3x3 convolution and the one or two 1x1 convolutions behind it: ConvArgs, then ChainArgs.
template <bool BF16, int NW>
__global__ __launch_bounds__(NW * 64) void conv_chain_kernel(const ConvArgs, const ChainArgs) {
  const ConstPtr src = (ConstPtr)__builtin_amdgcn_kernarg_segment_ptr();
  const ConvArgs p = conv_args_at(src);
  ChainArgs c = grab<ChainArgs>(src + sizeof(ConvArgs));
  c.w3 = in_memory(c.w3); c.bias3 = in_memory(c.bias3); c.res3 = in_memory(c.res3); c.y3 = in_memory(c.y3);
  c.w1 = in_memory(c.w1); c.bias1 = in_memory(c.bias1); c.y1 = in_memory(c.y1);
  __shared__ __align__(16) float lds[conv_chain_lds<BF16, NW>()];
  int mt, g;
  if (!conv_tile_of(p, (int)blockIdx.x, &mt, &g)) return;
  conv_chain_body<BF16, NW>(p, c, mt, lds);
  puts_done();
}
template __global__ void conv_chain_kernel<false, 8>(const ConvArgs, const ChainArgs);
template __global__ void conv_chain_kernel<true, 4>(const ConvArgs, const ChainArgs);

// FC, batch 1, behind a global average pooling of which the convolution has left sums.  Eight rows of the matrix to a workgroup, a wave each; the averages
// are made once per workgroup and lie in LDS, while the first weights are on their way.
template <bool BF16>
__global__ __launch_bounds__(kPooledRows * 64) void fc_pooled_kernel(const FcPooledArgs) {
  constexpr int VEC = BF16 ? 8 : 4, ES = BF16 ? 2 : 4, U = 8;  // U: loads of a lane in flight
  FcPooledArgs a = grab<FcPooledArgs>((ConstPtr)__builtin_amdgcn_kernarg_segment_ptr());
  args_in_memory(a);
  __shared__ __align__(16) float x[kPooledInputs];
  const int tid = threadIdx.x, lane = tid & 63, n = (int)blockIdx.x * kPooledRows + __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row = min(n, a.N - 1), nvec = a.K / VEC;  // (rows past the last one read it once more)
  const auto wrsrc = __builtin_amdgcn_make_buffer_rsrc((unsigned char*)const_cast<void*>(a.w) + (size_t)row * a.K * ES, 0, a.K * ES, 0x00027000);
  uint4 w[U];
  auto load = [&](int v) {
#pragma unroll
    for (int u = 0; u < U; ++u) w[u] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, (v + 64 * u) * 16, 0, 0));  // (past the row: zeros)
  };
  const float bias = a.bias[row];
  for (int k = 4 * tid; k < a.K; k += 256 * kPooledRows) {
    float4 t[kPooledTiles];
#pragma unroll
    for (int i = 0; i < kPooledTiles; ++i) {
      t[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (i < a.tiles) t[i] = *(const float4*)(a.x + (size_t)i * a.K + k);
    }
    if (k == 4 * tid) load(lane);
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int i = 0; i < 4; ++i) {  // (the order of gavgpool_group)
      s.x += t[i].x + t[i + 4].x; s.y += t[i].y + t[i + 4].y; s.z += t[i].z + t[i + 4].z; s.w += t[i].w + t[i + 4].w;
    }
    const float d = (float)a.pixels;
    s.x /= d; s.y /= d; s.z /= d; s.w /= d;
    if constexpr (BF16) {
      const uint32_t p = pack_bf16_rne(s.x, s.y), q = pack_bf16_rne(s.z, s.w);
      s = make_float4(__uint_as_float(p << 16), __uint_as_float(p & 0xffff0000u), __uint_as_float(q << 16), __uint_as_float(q & 0xffff0000u));
    }
    *(float4*)&x[k] = s;
  }
  if (4 * tid >= a.K) load(lane);
  __syncthreads();
  float acc4[4] = {0.f, 0.f, 0.f, 0.f};
  for (int v = lane; v < nvec + lane; v += 64 * U) {
    if (v != lane) load(v);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (v + 64 * u >= nvec) break;
      float wv[VEC];
      unpack<BF16>(w[u], wv);
      const float* const xv = x + (v + 64 * u) * VEC;
#pragma unroll
      for (int i = 0; i < VEC; i += 4) {
        const float4 q = *(const float4*)(xv + i);
        acc4[u & 3] = fmaf(wv[i], q.x, acc4[u & 3]); acc4[u & 3] = fmaf(wv[i + 1], q.y, acc4[u & 3]);
        acc4[u & 3] = fmaf(wv[i + 2], q.z, acc4[u & 3]); acc4[u & 3] = fmaf(wv[i + 3], q.w, acc4[u & 3]);
      }
    }
  }
  float acc = (acc4[0] + acc4[1]) + (acc4[2] + acc4[3]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if (lane == 0 && n < a.Ns) {
    const float v = n < a.N ? apply_act(acc + bias, a.act) : 0.f;  // (pad elements of the output vector are 0)
    if (a.out_f32) put((float*)a.y + n, v);
    else put_elem<BF16>(a.y, n, v);
  }
  puts_done();
}
template __global__ void fc_pooled_kernel<false>(const FcPooledArgs);
template __global__ void fc_pooled_kernel<true>(const FcPooledArgs);

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

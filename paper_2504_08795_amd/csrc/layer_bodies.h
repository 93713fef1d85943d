// What the kernels of several code objects run per tile: how a workgroup finds its convolution tile, the 32- and 16-pixel
// wave tiles, and the depthwise, pooling and FC layers.  (Device code.)
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace daris {

// Workgroup L of a convolution -> (pixel tile mt, weight group g = channel tile + n_tiles * K slice); false: nothing to do
// (padding).  Workgroups are handed to the 8 XCDs round-robin by linear id, and each XCD has its own L2: the mapping keeps
// all pixel tiles that read the same weights on one XCD (xmode 1: groups are a multiple of 8) or on 8/G of them (xmode 2),
// so that a weight byte is fetched from memory once per XCD that needs it instead of once per pixel tile.
__device__ __forceinline__ bool conv_tile_of(const ConvArgs& p, const int L, int* mt, int* g) {
  const int x = L & 7, q = L >> 3;
  if (p.xmode == 2) {  // G divides 8
    const int lr = 3 - __builtin_ctz(p.G);  // 8 / G tiles of a group side by side
    *g = x >> lr;
    *mt = (q << lr) + (x & ((1 << lr) - 1));
  } else {
    const int n = p.xmode == 1 ? q : L;
    const int d = p.mg_mt == kNoMagic ? n / p.MT : fast_div(n, p.mg_mt);
    *g = p.xmode == 1 ? d * 8 + x : d;
    *mt = n - d * p.MT;
  }
  return *g < p.G && *mt < p.MT;
}

// The arguments of a layer at `src`.
__device__ __forceinline__ ConvArgs conv_args_at(ConstPtr src) {
  ConvArgs p = grab<ConvArgs>(src);
  p.x = in_memory(p.x);
  p.w = in_memory(p.w);
  p.bias = in_memory(p.bias);
  p.res = in_memory(p.res);
  p.y = in_memory(p.y);
  p.ws = in_memory(p.ws);
  return p;
}
template <typename Args>
__device__ __forceinline__ void args_in_memory(Args& a) {
  a.x = in_memory(a.x);
  a.y = in_memory(a.y);
  if constexpr (!std::is_same<Args, PoolArgs>::value) {
    a.w = in_memory(a.w);
    a.bias = in_memory(a.bias);
  }
}
template <typename Args>
__device__ __forceinline__ Args args_at(ConstPtr src) {
  Args a = grab<Args>(src);
  if constexpr (std::is_same<Args, DwWindowArgs>::value || std::is_same<Args, PoolWindowArgs>::value) args_in_memory(a.a);
  else args_in_memory(a);
  return a;
}

// ---- tiles in plain fp32 arithmetic ---------------------------------------------------------------------------------
//
// An infinite operand, or parts that overflow where the fp32 product does not, leave the products in three parts as NaN or
// infinite, and pixels so small that their third part falls below the smallest bf16 number leave sums below 2^-103 short of
// bits.  A wave that finds its partial tile not finite, or all of it below 2^-103 (and not all of it 0), spoils the whole tile, so
// every thread of the workgroup meets a NaN in the sums that it reads anyway, and the workgroup walks its K slice a second time
// on the fp32 matrix instructions (plain_products).  What is not finite takes the second walk's sum, and so does all of a wave's tile that has nothing of 2^-103 and
// more that is finite; the other sums stay, so that a NaN or an infinity changes no sum but those that it is part of, whichever tile these lie in.  Nothing else in the launch depends on the data, so a launch in which every
// tile is taken twice is the longest there can be: the second walk, 8/3 of the first one's matrix time and with one chunk in
// flight, is bounded by the same K.
// The look at the partial tile is one instruction for two values, v_maximum3_f32 of their magnitudes, which keeps NaN.  A lane's
// largest magnitude times 2^-23 is denormal if it is below 2^-103 and not 0, so one test of its class finds all that is to be
// looked at closely: nothing that can be measured, where a second comparison costs 0.05 us a launch.  `tile` = the wave's
// partial tile in LDS, `words` floats a lane.
template <int N, typename Acc>
__device__ __forceinline__ bool out_of_range(const Acc (&acc)[N]) {
  constexpr int V = sizeof(Acc) / sizeof(float);
  float t[2] = {0.f, 0.f};
#pragma unroll
  for (int j = 0; j < N; ++j)
#pragma unroll
    for (int v = 0; v < V; v += 2)
      t[(v >> 1) & 1] = __builtin_elementwise_maximum(__builtin_elementwise_maximum(__builtin_fabsf(acc[j][v]), __builtin_fabsf(acc[j][v + 1])), t[(v >> 1) & 1]);
  const float largest = __builtin_elementwise_maximum(t[0], t[1]);
  constexpr int kNanInfDenormal = 0x283;  // signalling and quiet NaN, positive denormal, +infinity
  return __builtin_expect(__ballot(__builtin_amdgcn_classf(largest * 0x1p-23f, kNanInfDenormal)) != 0, 0) &&
         (__ballot(!(largest < INFINITY)) != 0 || __ballot(largest >= 0x1p-103f) == 0);
}
// Kernels that load real neighbours for the pixels of a tile that lie past the output keep these out of the test: nobody stores their sums, and
// one of ordinary size would keep a tile of small sums from being walked again.  Where lanes find their pixels in LDS by a place (conv_taps_body,
// conv_image_body), such a pixel is the place of zeros, chosen in a branch that whole tiles do not take, while the first loads are on their way.
// The 64 x 64 tiles, whose lanes have one place for several pixels, set the sums to 0 before the test: one comparison with a constant and one
// select a sum, behind such a branch; tiles of 32 pixels took 0.05 to 0.17 us longer that way.
// inside: how many of the block's pixels lie inside the output.
__device__ __forceinline__ void drop_pixels(f32x16& acc, const int inside) {
  const int left = inside - ((threadIdx.x & 63) >> 5) * 4;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = (v >> 2) * 8 + (v & 3) < left ? acc[v] : 0.f;
}
template <int N, typename Acc>
__device__ __forceinline__ void spoil_unless_in_range(const Acc (&acc)[N], float* const tile, const int words) {
  if (out_of_range(acc)) {
#pragma unroll 1
    for (int i = 0; i < words; ++i) tile[64 * i + (threadIdx.x & 63)] = __builtin_nanf("");
  }
}
// Which of a wave's sums the second walk replaces: all of a partial tile without a finite sum of 2^-103 and more, or those that are not finite.
template <typename Acc>
__device__ __forceinline__ bool all_small(const Acc& acc) {
  float largest = 0.f;
#pragma unroll
  for (int v = 0; v < (int)(sizeof(Acc) / sizeof(float)); ++v) {
    const float a = __builtin_fabsf(acc[v]);
    largest = a < INFINITY ? fmaxf(largest, a) : largest;
  }
  return __ballot(largest >= 0x1p-103f) == 0;
}
template <int N, typename Acc>
__device__ __forceinline__ bool all_small(const Acc (&acc)[N]) {
  bool small = true;
#pragma unroll
  for (int j = 0; j < N; ++j) small = all_small(acc[j]) && small;
  return small;
}
__device__ __forceinline__ float second(const bool small, const float first, const float again) {
  const float kept = small ? __builtin_nanf("") : first;
  const float sum = __builtin_fabsf(kept) < INFINITY ? kept : again;
  __builtin_amdgcn_sched_barrier(0);  // (one after the other: all comparisons first would take more scalar registers than there are)
  return sum;
}
template <typename Acc>
__device__ __forceinline__ void take_second(const bool small, const Acc& first, Acc& again) {
#pragma unroll
  for (int v = 0; v < (int)(sizeof(Acc) / sizeof(float)); ++v) again[v] = second(small, first[v], again[v]);
}
__device__ __forceinline__ bool spoiled(const float v) { return __ballot(__builtin_isnan(v)) != 0; }

// Pixel operand at k .. k + 3 (one filter tap, channel strides being multiples of four) of pixel m; MODE as in conv_wave_body.
template <int MODE>
__device__ __forceinline__ float4 pixel_quad(const ConvArgs& p, const DwFusedArgs& dwf, const int m, const int k) {
  const int y = fast_div(m, p.mg_wo), x = m - y * p.Wo;
  const int tap = MODE == 2 ? k >> 2 : fast_div(k, p.mg_cin), c = MODE == 2 ? 0 : k - tap * p.Cin;
  const int ky = fast_div(tap, p.mg_kw), kx = tap - ky * p.kw;
  const int iy = y * p.stride - p.pad + ky, ix = x * p.stride - p.pad + kx;
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (m >= p.M || ky >= p.kh || (unsigned)iy >= (unsigned)p.H || (unsigned)ix >= (unsigned)p.W) return v;
  if constexpr (MODE == 4) {
    v = *(const float4*)(dwf.bias + c);
#pragma unroll 1
    for (int t = 0; t < 9; ++t) {
      const int jy = iy * dwf.stride - 1 + t / 3, jx = ix * dwf.stride - 1 + t % 3;
      if ((unsigned)jy >= (unsigned)dwf.H || (unsigned)jx >= (unsigned)dwf.W) continue;
      const float4 in = *(const float4*)((const float*)p.x + (size_t)(jy * dwf.W + jx) * p.Cin + c), w = *(const float4*)((const float*)dwf.w + (size_t)t * p.Cin + c);
      v.x = fmaf(in.x, w.x, v.x); v.y = fmaf(in.y, w.y, v.y); v.z = fmaf(in.z, w.z, v.z); v.w = fmaf(in.w, w.w, v.w);
    }
    v.x = apply_act(v.x, dwf.act); v.y = apply_act(v.y, dwf.act); v.z = apply_act(v.z, dwf.act); v.w = apply_act(v.w, dwf.act);
  } else if constexpr (MODE == 2) {
    const float* const at = (const float*)p.x + (size_t)iy * p.W + ix;
    const size_t plane = (size_t)p.H * p.W;
    v.x = at[0];
    if (p.c_real > 1) v.y = at[plane];
    if (p.c_real > 2) v.z = at[2 * plane];
    if (p.c_real > 3) v.w = at[3 * plane];
  } else {
    v = *(const float4*)((const float*)p.x + (size_t)(iy * p.W + ix) * p.Cin + c);
  }
  return v;
}

// acc[i * TN + j] = the wave's partial tile of pixels m0 + R i .. and channel blocks nb0 + j over K steps [s0, s0 + nsteps), R = 32
// or 16.  The weights are put together from their parts (exact but for weights below 2^-110, see split8); a lane's eight k of a chunk go through the matrix
// pipe one at a time.
template <int MODE, int R, int TM, int TN, typename Acc>
__device__ __forceinline__ void plain_products(const ConvArgs& p, const DwFusedArgs& dwf, const int m0, const int nb0, const int s0, const int nsteps, Acc (&acc)[TM * TN]) {
  constexpr int CK = R == 16 ? 32 : 16;  // k of a chunk = two steps of the plan
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < TM * TN; ++i) acc[i] = Acc(0.f);
  const unsigned char* const wb = (const unsigned char*)p.w + (size_t)nb0 * (p.S >> 1) * 3072 + lane * 16;
#pragma unroll 1
  for (int c = s0 >> 1; c < (s0 + nsteps) >> 1; ++c) {
    float a[TM][8], b[TN][8];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      float w[3][8];
#pragma unroll
      for (int q = 0; q < 3; ++q) unpack<true>(*(const uint4*)(wb + ((size_t)j * (p.S >> 1) + c) * 3072 + q * 1024), w[q]);
#pragma unroll
      for (int e = 0; e < 8; ++e) b[j][e] = (w[2][e] + w[1][e]) + w[0][e];
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        int k = c * CK;
        if constexpr (MODE == 5 || MODE == 7) {  // chunks in the order (ky, 16 channels, kx) of three taps
          const int gk = c / 3 * CK, ky = fast_div(gk, p.mg_cin);
          k = (3 * ky + c % 3) * p.Cin + gk - ky * p.Cin;
        }
        int m = m0 + R * i + lane % R;
        if constexpr (MODE == 6) {  // two rows of 16 pixels, the first at m0
          const int x = m0 - fast_div(m0, p.mg_wo) * p.Wo + lane % 16;
          m = x < p.Wo ? m0 + (2 * i + lane % R / 16) * p.Wo + lane % 16 : p.M;
        }
        if constexpr (MODE == 7) {  // two rows of the image, from place m0 on (conv_block_body with POOL)
          const int s = m0 + lane % R;
          m = 2 * s < p.M ? s + (fast_div(s, p.mg_wo) + i) * p.Wo : p.M;
        }
        const float4 v = pixel_quad<MODE == 6 ? 2 : MODE == 7 ? 5 : MODE>(p, dwf, m, k + 8 * (lane / R) + 4 * h);
        a[i][4 * h] = v.x; a[i][4 * h + 1] = v.y; a[i][4 * h + 2] = v.z; a[i][4 * h + 3] = v.w;
      }
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          if constexpr (R == 16) acc[i * TN + j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], b[j][e], acc[i * TN + j], 0, 0, 0);
          else acc[i * TN + j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], b[j][e], acc[i * TN + j], 0, 0, 0);
        }
  }
}

// ---- wave-tile implicit GEMM ---------------------------------------------------------------------------------------
//
// For the small-M, deep-K convolutions of batch-1 inference an output tile shared through LDS buys nothing: there
// are too few tiles to fill a partition, so K has to be split anyway.  Here one wave owns a 32 x (32*TN) output
// tile over a slice of K and feeds the MFMA straight from registers: lane (i, h) loads the 16 bytes of pixel
// m0+i at k = step*KS + h*VEC.. from the NHWC input and, per channel block, 16 bytes of weights that were packed
// at registration in exactly this order ([channel block][step][lane][16 B]: one fully coalesced 1 KiB read per
// step, consecutive steps consecutive in memory).  No barrier and no LDS in the K loop; D steps are in flight.
// The NW waves of a workgroup split the K slice of the workgroup; their partial tiles are summed through LDS in
// wave order.  With splitk > 1 several workgroups share one tile, split K as well and write partial sums to the workspace,
// which splitk_reduce_kernel adds in z order (a device-wide fence per workgroup for an in-kernel reduction was
// measured to cost several times the extra launch).
//
// The pixels are requested before the weights: loads return in order, and what the pixels pass through on their way to the
// matrix pipe takes longer (0.25 us per launch the other way round).
// What a wave tile's launch does once the K loop is over: the partial tiles of the NW waves are summed through LDS in wave
// order and each sum gets bias, residual and activation.  R = 32 or 16 pixels, channel blocks of the same size.  Works on quads of
// consecutive channels: quad q of the tile = elements 4q..4q+3 = lanes l..l+3 of one accumulator row (j, v), i.e. one pixel
// (place()) and channels R*(nb0+j) + l%R .. +3.  A thread's quads q = tid + r*NT all have the same l, so it needs the bias of
// one channel quad per channel block; that and the residual are fetched ahead of the sums (when this launch applies them itself).
template <int R>
using WaveAcc = typename std::conditional<R == 32, f32x16, f32x4>::type;
// BUFFER: everything goes through buffer descriptors, which give 0 past the end and drop what is stored there, so that nothing is
// conditional and the compiler can count the loads.  They hold the whole tensors, below 2 GiB, or (LARGE) the tile's pixels.
// TM = 2 (with TN = 1): two blocks of pixels in place of two of channels.
template <bool BF16, int R, int TN, int NW, bool BUFFER, bool LARGE = false, int TM = 1>
struct WaveEpilogue {
  static_assert(TM == 1 || (R == 16 && TN == 1 && !LARGE), "blocks of pixels or of channels");
  static constexpr int ES = BF16 ? 2 : 4, NT = NW * 64, V = R * R / 64, TILE = TM * TN * R * R;  // V: accumulator rows of a block
  static constexpr int QUADS = TILE / 4, RQ = (QUADS + NT - 1) / NT;  // quads of the tile, of a thread
  static constexpr int NB = RQ == 1 ? 1 : TN;
  using ResVec = typename std::conditional<BF16, uint2, uint4>::type;
  static constexpr int kOutside = (int)0x80000000;  // an offset past the end of any tensor
  float4 bias_j[NB];
  ResVec res_pre[RQ];
  int at[RQ];  // BUFFER: byte offset of the quad in the output and in the residual operand (LARGE: from the tile's first pixel on)
  bool own_epilogue, use_res;

  // channel block, pixel and first channel of the quad that starts at tile element e = (j*V + v)*64 + lane
  __device__ __forceinline__ void place(const int e, const int m0, const int nb0, int* j, int* mm, int* n) const {
    const int v = (e >> 6) % V, l = e & 63, block = (e >> 6) / V;
    *j = TM == 1 ? block : 0;
    *mm = m0 + (TM == 1 ? 0 : block * R) + (R == 32 ? (v >> 2) * 8 + (l >> 5) * 4 + (v & 3) : (l >> 4) * 4 + v);
    *n = (nb0 + *j) * R + l % R;
  }
  // LARGE: `t`, of the output's shape, from the tile's first pixel on
  __device__ __forceinline__ static void* from_tile(const ConvArgs& p, const void* t, const int m0) {
    return (unsigned char*)const_cast<void*>(t) + (size_t)(uint32_t)m0 * (uint32_t)(p.Cout * ES);
  }
  __device__ __forceinline__ void fetch(const ConvArgs& p, const int m0, const int nb0, const int tid) {
    own_epilogue = p.splitk == 1;
    use_res = own_epilogue && p.res != nullptr;
    const auto brsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.bias), 0, BUFFER ? p.Cout * 4 : 0, 0x00027000);
    const auto rrsrc = __builtin_amdgcn_make_buffer_rsrc(LARGE ? from_tile(p, p.res, m0) : const_cast<void*>(p.res), 0, BUFFER && use_res ? (LARGE ? min(R, p.M - m0) : p.M) * p.Cout * ES : 0, 0x00027000);
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      int j, mm, n;
      place(4 * tid, m0, nb0, &j, &mm, &n);
      if (NB > 1) n += (k - j) * R;
      if constexpr (BUFFER) bias_j[k] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(brsrc, n * 4, 0, 0));
      else bias_j[k] = (n < p.Cout) ? *(const float4*)(p.bias + n) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int r = 0; r < RQ; ++r) {
      res_pre[r] = ResVec();
      const int e = 4 * (tid + r * NT);
      int j, mm, n;
      place(e, m0, nb0, &j, &mm, &n);
      const bool ok = (QUADS % NT == 0 || e < TILE) && mm < p.M && n < p.Cout;
      if constexpr (BUFFER) {
        at[r] = ok ? ((LARGE ? mm - m0 : mm) * p.Cout + n) * ES : kOutside;
        if constexpr (BF16) res_pre[r] = __builtin_bit_cast(ResVec, __builtin_amdgcn_raw_buffer_load_b64(rrsrc, at[r], 0, 0));
        else res_pre[r] = __builtin_bit_cast(ResVec, __builtin_amdgcn_raw_buffer_load_b128(rrsrc, at[r], 0, 0));
      } else if (use_res && ok) {
        res_pre[r] = *(const ResVec*)((const unsigned char*)p.res + ((size_t)mm * p.Cout + n) * ES);
      }
    }
  }

  // MODE as in conv_wave_body; acc = the wave's partial tile over K steps [sbeg, sbeg + nsteps); kNoWalk: there is no second walk.
  // KEEP: the outputs go to `kept` in LDS, rows of kept_row bytes (zeros past the last pixel), instead of to memory.
  static constexpr int kNoWalk = -1;
  template <int MODE, bool KEEP = false>
  __device__ __forceinline__ void finish(const ConvArgs& p, const DwFusedArgs& dwf, WaveAcc<R> (&acc)[TM * TN], float* const red, const int m0, const int nb0, const int zi,
                                         const int sbeg, const int nsteps, unsigned char* const kept = nullptr, const int kept_row = 0) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto park = [&]() {
#pragma unroll
      for (int j = 0; j < TM * TN; ++j)
#pragma unroll
        for (int v = 0; v < V; ++v) red[wave * TILE + (j * V + v) * 64 + lane] = acc[j][v];
    };
    float4 sums[RQ];
    auto add_up = [&]() {
#pragma unroll
      for (int r = 0; r < RQ; ++r) {
        const int e = 4 * (tid + r * NT);
        if (QUADS % NT != 0 && wave >= QUADS / 64) {  // (the waves past the tile)
          sums[r] = make_float4(0.f, 0.f, 0.f, 0.f);
          if (!BF16) sums[r].x = red[lane % NW * TILE + lane];  // ... look whether one of the partial tiles is spoiled
          continue;
        }
        sums[r] = *(const float4*)&red[e];
#pragma unroll
        for (int w = 1; w < NW; ++w) {
          const float4 t = *(const float4*)&red[w * TILE + e];
          sums[r].x += t.x; sums[r].y += t.y; sums[r].z += t.z; sums[r].w += t.w;
        }
      }
    };
    park();
    if constexpr (!BF16 && MODE != kNoWalk) {
      spoil_unless_in_range(acc, red + wave * TILE, V * TM * TN);
    }
    __syncthreads();
    add_up();
    if constexpr (!BF16 && MODE != kNoWalk) {
      if (__builtin_expect(spoiled(sums[0].x), 0)) {  // every thread of the workgroup or none (out of the way: a launch fetches its code anew, and a longer path costs 0.2 us)
        __syncthreads();
        park();
        const bool small = all_small(acc);
        plain_products<MODE, R, TM, TN>(p, dwf, m0, nb0, sbeg, nsteps, acc);
#pragma unroll
        for (int j = 0; j < TM * TN; ++j)
#pragma unroll
          for (int v = 0; v < V; ++v) {
            float& at = red[wave * TILE + (j * V + v) * 64 + lane];
            at = second(small, at, acc[j][v]);
          }
        __syncthreads();
        add_up();
      }
    }
    if (!KEEP && !own_epilogue) {  // partial sums of this K slice; splitk_reduce_kernel finishes the layer
#pragma unroll
      for (int r = 0; r < RQ; ++r) {
        const int e = 4 * (tid + r * NT);
        int j, mm, n;
        place(e, m0, nb0, &j, &mm, &n);
        if ((QUADS % NT == 0 || e < TILE) && mm < p.M && n < p.Cout) put(p.ws + (size_t)zi * p.M * p.Cout + (size_t)mm * p.Cout + n, sums[r]);
      }
      return;
    }
    // All quads are finished before the first is stored: loads and stores are counted together, so a quad that waited for its
    // residual behind a store would wait for the store's way to memory as well, 0.5 us each (3136 x 256 x 64 in bf16, four
    // quads a thread: 1.3 us of a launch of 4.5).
    float val[4 * RQ];
#pragma unroll
    for (int r = 0; r < RQ; ++r) {
      const int j = ((4 * (tid + r * NT)) >> 6) / V;
      float4 b = bias_j[0];  // component-wise select: indexing the array with a run-time j would move it out of registers
      if (NB == 2) {
        const bool hi = j != 0;
        b.x = hi ? bias_j[NB - 1].x : b.x; b.y = hi ? bias_j[NB - 1].y : b.y;
        b.z = hi ? bias_j[NB - 1].z : b.z; b.w = hi ? bias_j[NB - 1].w : b.w;
      }
      val[4 * r] = sums[r].x + b.x; val[4 * r + 1] = sums[r].y + b.y; val[4 * r + 2] = sums[r].z + b.z; val[4 * r + 3] = sums[r].w + b.w;
    }
    if (use_res) {
#pragma unroll
      for (int r = 0; r < RQ; ++r) {
        const ResVec rv = res_pre[r];
        if constexpr (BF16) {
          val[4 * r] += __uint_as_float(rv.x << 16); val[4 * r + 1] += __uint_as_float(rv.x & 0xffff0000u);
          val[4 * r + 2] += __uint_as_float(rv.y << 16); val[4 * r + 3] += __uint_as_float(rv.y & 0xffff0000u);
        } else {
          val[4 * r] += __uint_as_float(rv.x); val[4 * r + 1] += __uint_as_float(rv.y);
          val[4 * r + 2] += __uint_as_float(rv.z); val[4 * r + 3] += __uint_as_float(rv.w);
        }
      }
    }
    // (only where plans ask for it: in the kernels without descriptors, 10900 x 96 x 16 in bf16 on 64 CUs went from 4.8 to 5.3 us for it)
    constexpr bool SUMS = BUFFER && !LARGE && !KEEP && MODE != kNoWalk;
    apply_act(val, SUMS ? p.act & kActMask : p.act);
    if (SUMS && __builtin_expect(p.act & kActSumPixels, 0)) {  // the sums of the tile's outputs over its pixels, for the global average behind the layer
      __syncthreads();  // (every thread has read its partial sums)
#pragma unroll
      for (int r = 0; r < RQ; ++r) {
        const int e = 4 * (tid + r * NT);
        int j, mm, n;
        place(e, m0, nb0, &j, &mm, &n);
        const bool in = mm < p.M;
        float4 v;
        v.x = in ? val[4 * r] : 0.f; v.y = in ? val[4 * r + 1] : 0.f; v.z = in ? val[4 * r + 2] : 0.f; v.w = in ? val[4 * r + 3] : 0.f;
        if constexpr (BF16) {
          const uint32_t a = pack_bf16_rne(v.x, v.y), b = pack_bf16_rne(v.z, v.w);
          v = make_float4(__uint_as_float(a << 16), __uint_as_float(a & 0xffff0000u), __uint_as_float(b << 16), __uint_as_float(b & 0xffff0000u));
        }
        if (QUADS % NT == 0 || e < TILE) *(float4*)&red[e] = v;
      }
      __syncthreads();
      const int c = threadIdx.x % R, block = threadIdx.x / R, n = (nb0 + (TM == 1 ? block : 0)) * R + c;
      if (block < TM * TN && n < p.Cout) {
        const float* const from = red + block * (R * R) + c;
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < R; ++i) {  // in the order of the pixels
          const int v = R == 32 ? (i >> 3) * 4 + (i & 3) : i & 3, lanes = R == 32 ? (i >> 2 & 1) * 32 : (i >> 2) * 16;
          s += from[v * 64 + lanes];
        }
        const int mt = m0 / R + (TM == 1 ? 0 : block);
        if (mt * R < p.M) put((float*)p.y + (size_t)mt * p.Cout + n, s);
      }
      return;
    }
    ResVec out[RQ];
#pragma unroll
    for (int r = 0; r < RQ; ++r) {
      const float* const v = val + 4 * r;
      if constexpr (BF16) {
        out[r].x = pack_bf16_rne(v[0], v[1]);
        out[r].y = pack_bf16_rne(v[2], v[3]);
      } else {
        out[r] = make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3]));
      }
    }
    if constexpr (KEEP) {
      static_assert(BUFFER && QUADS % NT == 0, "every thread has quads, and their places");
#pragma unroll
      for (int r = 0; r < RQ; ++r) {
        int j, mm, n;
        place(4 * (tid + r * NT), m0, nb0, &j, &mm, &n);
        const bool in = at[r] != kOutside;
        ResVec v = out[r];
        v.x = in ? v.x : 0u; v.y = in ? v.y : 0u;
        if constexpr (!BF16) { v.z = in ? v.z : 0u; v.w = in ? v.w : 0u; }
        *(ResVec*)(kept + (mm - m0) * kept_row + n * ES) = v;
      }
      return;
    }
    const auto yrsrc = __builtin_amdgcn_make_buffer_rsrc(LARGE ? from_tile(p, p.y, m0) : p.y, 0, BUFFER ? (LARGE ? min(R, p.M - m0) : p.M) * p.Cout * ES : 0, 0x00027000);
#pragma unroll
    for (int r = 0; r < RQ; ++r) {
      if constexpr (BUFFER) {
        put_at(yrsrc, at[r], out[r]);
      } else {
        const int e = 4 * (tid + r * NT);
        int j, mm, n;
        place(e, m0, nb0, &j, &mm, &n);
        if ((QUADS % NT == 0 || e < TILE) && mm < p.M && n < p.Cout) put((unsigned char*)p.y + ((size_t)mm * p.Cout + n) * ES, out[r]);
      }
    }
  }
};

template <bool BF16, int TN, int NW, int MODE>
constexpr int conv_wave_lds() {  // floats of LDS
  return MODE == 4 && NW * 32 * 5 * 4 > NW * TN * 1024 ? NW * 32 * 5 * 4 : NW * TN * 1024;
}
template <bool BF16, int TN, int NW, int MODE, int DC>
__device__ __forceinline__ void conv_wave_body(const ConvArgs& p, const int mt, const int g, float* const red, const DwFusedArgs& dwf) {
  // MODE 0 (bf16): Cin a multiple of KS; 1: any Cin; 2: the network input itself, fp32 [C][H][W]; 4: a 1x1 convolution whose
  // input is the output of a 3x3 depthwise convolution that is never stored: the rows are computed here from the depthwise
  // layer's input (p.x) and weights (dwf).  (3: conv_rows_body)
  // fp32: two K steps of 8 make one chunk of 16, the depth of the bf16 matrix instruction that takes the operands' three
  // parts (split8); the plan cuts K in whole chunks, the weights are stored as [channel block][chunk][part][lane][16 B].
  constexpr bool ALIGNED = MODE == 0;
  static_assert(BF16 || MODE != 0, "fp32 locates its quads of channels in closed form whatever Cin is");
  constexpr bool STAGED = MODE == 4;
  constexpr int ES = BF16 ? 2 : 4;
  constexpr int VEC = 16 / ES;
  constexpr int KS = 2 * VEC;
  constexpr int NT = NW * 64;
  constexpr int TILE = TN * 1024;
  constexpr int D = 4;                  // bf16: K steps in flight
  // (DC: fp32: chunks of weights in flight)
  constexpr int STAGE_V = 32 * 5;  // 16-byte vectors of one wave's staging buffer: 32 pixels x (4 pieces + 1 pad)
  static_assert(TN == 1 || TN == 2, "the epilogue selects between at most two channel blocks");
  static_assert((TILE / 4) % NT == 0 || NT % (TILE / 4) == 0, "tile / thread mismatch");

  if (p.wave_prio) __builtin_amdgcn_s_setprio(3);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: keeps the K loop's control flow scalar
  const int li = lane & 31, lh = lane >> 5;
  const int zi = p.splitk == 1 ? 0 : g / p.NTn;
  const int m0 = mt * 32, nb0 = (g - zi * p.NTn) * TN;

  const int s_wg0 = zi * p.sz;
  const int s_wg1 = min(s_wg0 + p.sz, p.S);
  const int sbeg = min(s_wg0 + wave * p.sw, s_wg1);
  const int nsteps = min(sbeg + p.sw, s_wg1) - sbeg;

  const unsigned char* xb = (const unsigned char*)p.x;
  const int m = m0 + li;
  const bool a_ok = m < p.M;
  const int oy = fast_div(m, p.mg_wo), ox = m - oy * p.Wo;
  const int iy0 = oy * p.stride - p.pad, ix0 = ox * p.stride - p.pad;
  // Walk over k = (tap, ci).  ALIGNED (Cin a multiple of KS): both lane halves are always in the same tap, so the
  // walk state (ky, kx, ci) is wave-uniform and lives in scalars; a lane adds its half's offset lh*VEC, a step
  // inside a tap only advances the pointer and a new tap recomputes pointer and validity.  Otherwise (the padded
  // network input, Cin < KS, or Cin not a multiple of KS) each lane derives tap and channel of its vector from the
  // step number in closed form: no lane-dependent branch, so the loads stay unconditional and pipelined.
  int kcur = sbeg * KS;  // k of the next step to load (scalar)
  int tap = fast_div(kcur, p.mg_cin);
  int ci = kcur - tap * p.Cin;
  int ky = fast_div(tap, p.mg_kw), kx = tap - ky * p.kw;
  bool a_valid;
  const unsigned char* ap;
  auto enter_tap = [&]() {
    const int iy = iy0 + ky, ix = ix0 + kx;
    a_valid = a_ok && ky < p.kh && (unsigned)iy < (unsigned)p.H && (unsigned)ix < (unsigned)p.W;
    ap = xb + ((size_t)(a_valid ? iy * p.W + ix : 0) * p.Cin + ci + lh * VEC) * ES;  // always a valid address
  };
  // MODE 2 reads the caller's fp32 [C][H][W] input directly (no separate layout conversion launch): the padded channel
  // count equals VEC, so a lane's vector is one filter tap, gathered as four scalar loads from the channel planes.
  // Planes beyond the real channel count repeat the last real one; their weights are zero.
  // The loads go through a buffer descriptor: one 32-bit offset per tap for all planes, and 0 comes back where the tap lies
  // outside the image, which takes half of the vector instructions out of the gather (12544 x 64 x 196
  // on 128 CUs: fp32 11.2 -> 10.6 us, bf16 8.3 -> 7.5; 50176 x 64 x 27: 12.6 -> 12.1).
  const int plane = p.H * p.W * 4;
  const auto irsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.x), 0, MODE == 2 ? p.c_real * plane : 0, 0x00027000);
  const int po1 = min(1, p.c_real - 1) * plane, po2 = min(2, p.c_real - 1) * plane, po3 = min(3, p.c_real - 1) * plane;
  auto tap_pixels = [&](bool ok, int iy, int ix) {  // MODE 2
    const int o = ok ? (iy * p.W + ix) * 4 : -4;
    return make_uint4(__builtin_amdgcn_raw_buffer_load_b32(irsrc, o, 0, 0), __builtin_amdgcn_raw_buffer_load_b32(irsrc, o, po1, 0),
                      __builtin_amdgcn_raw_buffer_load_b32(irsrc, o, po2, 0), __builtin_amdgcn_raw_buffer_load_b32(irsrc, o, po3, 0));
  };
  int tap_y = 0, tap_x = 0;
  auto locate = [&]() {  // !ALIGNED: this lane's vector of step kcur
    const int k = kcur + lh * VEC;
    const int t = MODE == 2 ? k / VEC : fast_div(k, p.mg_cin), c = k - t * p.Cin;
    const int y = fast_div(t, p.mg_kw), x = t - y * p.kw;
    const int iy = iy0 + y, ix = ix0 + x;
    a_valid = a_ok && y < p.kh && (unsigned)iy < (unsigned)p.H && (unsigned)ix < (unsigned)p.W;
    if (MODE == 2) {
      tap_y = iy;
      tap_x = ix;
    } else ap = xb + ((size_t)(a_valid ? iy * p.W + ix : 0) * p.Cin + c) * ES;
  };
  if (ALIGNED) enter_tap();
  const unsigned char* wptr[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j)
    wptr[j] = BF16 ? (const unsigned char*)p.w + (((size_t)(nb0 + j) * p.S + sbeg) * 64 + lane) * 16
                   : (const unsigned char*)p.w + ((((size_t)(nb0 + j) * p.S + sbeg) >> 1) * 192 + lane) * 16;

  uint4 ar[D], br[D][TN];
  bool av[D];  // validity of slot d's A vector; the blanking is applied when the slot is consumed, so that a load's
               // result is not touched (and not waited for) until D-1 later steps have been issued
  auto load = [&](int d) {
    if (!ALIGNED) locate();
    if (MODE == 2) ar[d] = tap_pixels(a_valid, tap_y, tap_x);
    else ar[d] = *(const uint4*)ap;
    av[d] = MODE == 2 || a_valid;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      br[d][j] = *(const uint4*)wptr[j];
      wptr[j] += 1024;
    }
    if (ALIGNED) {
      ci += KS;
      if (ci >= p.Cin) {  // wave-uniform
        ci -= p.Cin;
        if (++kx == p.kw) { kx = 0; ++ky; }
        enter_tap();
      } else {
        ap += KS * ES;
      }
    } else {
      kcur += KS;
    }
  };

  WaveEpilogue<BF16, 32, TN, NW, false> fin;
  fin.fetch(p, m0, nb0, tid);

  f32x16 acc[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;

  auto mma = [&](uint4 a4, const uint4* b) {
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[j] = mfma_bf16(a4, b[j], acc[j]);
  };
  // fp32: one chunk of 16 k.  The terms go in from the smallest to the largest; the TN accumulators alternate so that
  // consecutive instructions are independent.
  uint4 bw[DC][TN][3];
  auto load_wc = [&](int d) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
#pragma unroll
      for (int q = 0; q < 3; ++q) bw[d][j][q] = *(const uint4*)(wptr[j] + q * 1024);
      wptr[j] += 3072;
    }
  };
  auto mma_chunk = [&](const uint4& lo, const uint4& hi, int d) {
    const Split8 a = split8(lo, hi);
    constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
    for (int t = 0; t < 6; ++t)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[j] = mfma_bf16(a.p[PA[t]], bw[d][j][PB[t]], acc[j]);
  };
  auto compute = [&](int d) {
    uint4 a4 = keep_if(av[d], ar[d]);
    if (MODE == 2 && BF16) {  // four fp32 channels -> the 8-channel bf16 vector of the tap (same rounding as the conversion kernel)
      a4.x = pack_bf16_rne(__uint_as_float(a4.x), __uint_as_float(a4.y));
      a4.y = pack_bf16_rne(__uint_as_float(a4.z), __uint_as_float(a4.w));
      a4.z = 0u;
      a4.w = 0u;
    }
    mma(a4, br[d]);
  };

  // Software pipeline, D steps deep.  Every load in the prologue and in the steady-state loop is unconditional and
  // the loop is straight-line (compute slot d, refill slot d), so the compiler can count the loads in flight and
  // wait only for the oldest slot.  Refills past the end of the wave's K slice fetch valid memory that is never used
  // (the weight buffer carries D KiB of slack; the A pointer always points into the input); only the computes of the
  // ragged tail are conditional.
  if constexpr (!STAGED && !BF16) {
    // register-fed fp32: a lane's eight k of a chunk are two quads, each inside one filter tap (channel strides are
    // multiples of four), located from the chunk number in closed form
    uint4 aq[DC][2];
    bool aqv[DC][2];
    kcur += lh * 8;
    auto load_c = [&](int d) {
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int k = kcur + 4 * e;
        const int t = MODE == 2 ? k / VEC : fast_div(k, p.mg_cin), c = k - t * p.Cin;
        const int y = fast_div(t, p.mg_kw), x = t - y * p.kw;
        const int iy = iy0 + y, ix = ix0 + x;
        const bool v = a_ok && y < p.kh && (unsigned)iy < (unsigned)p.H && (unsigned)ix < (unsigned)p.W;
        if (MODE == 2) aq[d][e] = tap_pixels(v, iy, ix);
        else aq[d][e] = *(const uint4*)(xb + ((size_t)(v ? iy * p.W + ix : 0) * p.Cin + (v ? c : 0)) * ES);  // always a valid address
        aqv[d][e] = MODE == 2 || v;
      }
      load_wc(d);
      kcur += 16;
    };
    auto compute_c = [&](int d) { mma_chunk(keep_if(aqv[d][0], aq[d][0]), keep_if(aqv[d][1], aq[d][1]), d); };
    const int nch = nsteps >> 1;
#pragma unroll
    for (int d = 0; d < DC; ++d) load_c(d);
    int done = 0;
    for (; done + DC <= nch; done += DC) {
#pragma unroll
      for (int d = 0; d < DC; ++d) {
        compute_c(d);
        load_c(d);
      }
    }
#pragma unroll
    for (int d = 0; d < DC; ++d)
      if (done + d < nch) compute_c(d);
  } else if constexpr (!STAGED) {
#pragma unroll
    for (int d = 0; d < D; ++d) load(d);
    int done = 0;
    for (; done + D <= nsteps; done += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        compute(d);
        load(d);
      }
    }
#pragma unroll
    for (int d = 0; d < D; ++d)
      if (done + d < nsteps) compute(d);
  } else {
    // The rows of a chunk of two K steps are computed where conv_rows_body would have loaded them, and pass through the wave's own
    // corner of LDS in the same way.
    uint4* const st = reinterpret_cast<uint4*>(red) + wave * STAGE_V;
    const int piece = lane & 3, prow = lane >> 2;
    auto load_w = [&](int d) {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        br[d][j] = *(const uint4*)wptr[j];
        wptr[j] += 1024;
      }
    };
    // rows in the wave's buffer -> MFMA order -> two K steps against the weights of chunk slot cs (bf16: of the pipeline
    // slots 2 cs, 2 cs + 1)
    auto exchange_and_mma = [&](int cs) {
      const int d0 = 2 * cs;
      // lanes exchange data through the wave's buffer: order the accesses of the whole wave, not only of each lane
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      uint4 a4[2];
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2) a4[s2] = st[li * 5 + (BF16 ? 2 * s2 + lh : 2 * lh + s2)];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      if constexpr (BF16) {
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          mma(a4[s2], br[d0 + s2]);
          load_w(d0 + s2);
        }
      } else {
        mma_chunk(a4[0], a4[1], cs);
        __builtin_amdgcn_sched_barrier(0);  // the refill takes over the registers of the slot just used (64 fewer in all)
        load_wc(cs);
      }
    };
    constexpr int CS = BF16 ? 2 : DC;  // chunks of weights in flight
    auto load_w_all = [&]() {
      if constexpr (BF16) {
#pragma unroll
        for (int d = 0; d < D; ++d) load_w(d);
      } else {
#pragma unroll
        for (int d = 0; d < DC; ++d) load_wc(d);
      }
    };
    const int nchunks = nsteps >> 1;
    // The 1x1 convolution's input row of pixel (y, x), channels c..c+VEC-1, is the depthwise layer's output there:
    // act(bias[c] + sum over the 3x3 taps inside the image, in (ky, kx) order, of in[y*stride-1+ky][x*stride-1+kx][c] * w[tap][c]),
    // accumulated with fused multiply-adds in exactly the order of dwconv_kernel, then rounded to the element type as a
    // stored tensor would be.  A lane computes the 16-byte piece it would otherwise have loaded.
    const unsigned char* dww = (const unsigned char*)dwf.w;
    int poff[2][9];     // element offset of each tap's input pixel (0 where the tap is outside: the value is not used)
    unsigned vmask[2];  // bit t: tap t of this lane's pixel lies inside the image
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int mj = m0 + 16 * j + prow;
      const bool okj = mj < p.M;
      const int y = fast_div(mj, p.mg_wo), x = mj - y * p.Wo;
      vmask[j] = 0u;
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const int iy = y * dwf.stride - 1 + t / 3, ix = x * dwf.stride - 1 + t % 3;
        const bool v = okj && (unsigned)iy < (unsigned)dwf.H && (unsigned)ix < (unsigned)dwf.W;
        poff[j][t] = v ? (iy * dwf.W + ix) * p.Cin : 0;
        vmask[j] |= v ? (1u << t) : 0u;
      }
    }
    int cch = sbeg * KS;  // first channel of the wave's next chunk (wave-uniform)
    uint4 xv[2][9], wv[9];
    float4 bv[VEC / 4];
    auto dw_issue = [&]() {  // loads of the chunk at cch (bf16 past the end of the slice: the last chunk of the tensor once more, never used)
      const int c = min(cch, p.Cin - 2 * KS) + piece * VEC;
#pragma unroll
      for (int t = 0; t < 9; ++t) wv[t] = *(const uint4*)(dww + ((size_t)t * p.Cin + c) * ES);
#pragma unroll
      for (int q = 0; q < VEC / 4; ++q) bv[q] = *(const float4*)(dwf.bias + c + 4 * q);
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int t = 0; t < 9; ++t) xv[j][t] = *(const uint4*)(xb + ((size_t)poff[j][t] + c) * ES);
      cch += 2 * KS;
    };
    auto dw_value = [&](int j) -> uint4 {
      float acc[VEC];
#pragma unroll
      for (int q = 0; q < VEC / 4; ++q) {
        acc[4 * q] = bv[q].x; acc[4 * q + 1] = bv[q].y; acc[4 * q + 2] = bv[q].z; acc[4 * q + 3] = bv[q].w;
      }
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        float xf[VEC], wf[VEC];
        unpack<BF16>(xv[j][t], xf);
        unpack<BF16>(wv[t], wf);
        const bool v = (vmask[j] >> t) & 1u;
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[i] = v ? fmaf(xf[i], wf[i], acc[i]) : acc[i];
      }
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[i] = apply_act(acc[i], dwf.act);
      return pack<BF16>(acc);
    };
    // more: another chunk follows, whose operands travel while this one goes through the matrix pipe.  Past the last chunk fp32 requests
    // no pixels, taps or biases (the weights' refill, three loads from the slack behind them, stays): 28 loads of the CU's vector memory unit that a wave of one to three chunks pays for (12544 x 16 x 32 6.2 -> 5.05 us, 3136 x
    // 24 x 96 6.33 -> 6.27, 3136 x 24 x 144 7.05 -> 6.88 on 128 CUs).  bf16, whose chunks go in twos, takes 70 registers more that way.
    auto chunk_dw = [&](int cs, bool more) {
#pragma unroll
      for (int j = 0; j < 2; ++j) st[(16 * j + prow) * 5 + piece] = dw_value(j);
      if (BF16 || more) dw_issue();
      exchange_and_mma(cs);
    };
    if (BF16 || nchunks > 0) {
      dw_issue();
      load_w_all();
    }
    int c = 0;
    for (; c + CS <= nchunks; c += CS) {
      chunk_dw(0, c + 1 < nchunks);
      if constexpr (CS == 2) chunk_dw(1, c + 2 < nchunks);
    }
    if (CS == 2 && c < nchunks) chunk_dw(0, false);
    __syncthreads();  // the partial tiles below reuse the LDS of every wave's staging buffer
  }

  fin.template finish<MODE>(p, dwf, acc, red, m0, nb0, zi, sbeg, nsteps);
}

// ---- wave tiles whose pixels are whole 64-byte rows (gather mode 3) ---------------------------------------------------------
//
// R = 32: 32 pixels x (32 * TN) channels per wave on v_mfma_f32_32x32x16_bf16.  R = 16: 16 pixels x (16 * TN) channels on
// v_mfma_f32_16x16x32_bf16, for layers with few output pixels and many channels (the 14x14 and 7x7 stages of a ResNet): these
// have too few 32 x 32 tiles to fill a partition, and would have to split K across workgroups and sum the partial tiles in
// a second launch; at the same matrix rate there are two to four times as many 16 x 16 tiles, K is split only among the
// NW waves of a workgroup, and the reduction launch disappears.
//
// A load instruction is served 64 bytes per cycle only when four neighbouring lanes read one 64-byte segment; with every lane in
// a different pixel (a different cache line) the pixel operand costs four times the cycles of the same bytes of weights.  So a
// wave fetches whole rows of 64 bytes (lane = (pixel, 16-byte piece)), parks them in its own corner of LDS, and reads them back
// in MFMA order.  No workgroup barrier is involved: the buffer is private to the wave.  A chunk, what goes through together, is
// two K steps: one row of each of 32 pixels, or two consecutive ones of each of 16.
// R = 32: lane (i, h) of a fragment holds pixel i and k = 8 h .. 8 h + 7 of a step (bf16) or of the chunk (fp32).
// R = 16: lane (i, q) holds pixel i and k = 8 q .. 8 q + 7 of a step (bf16) or of the chunk (fp32).
// Weights come in the same order: [channel block of R][step][lane][16 B] in bf16, [channel block of R][chunk][part][lane][16 B] in
// fp32, whose plan cuts K in whole chunks.
//
// A wave has one or two others on its SIMD and one to twenty chunks to walk, and what bounds the walk is the vector memory unit, which
// takes about twenty cycles for every load instruction of the CU, whether its data are used or not.  So nothing is loaded that is not
// used: DC chunks of rows and weights are in flight, and refills stop with the last chunk of the slice.  Which slot is refilled and
// which is the last one is known at compile time on every path (rows_pipeline), so that the compiler waits for one chunk and not for
// those behind it.  Rows outside the image are offsets past the end of a buffer descriptor, which returns 0 (an instruction whose
// lanes are all outside takes its twenty cycles too, so refills past the end cannot be left to it).  Against unconditional
// refills, on 128 CUs: fp32 3136 x 64 x 576 7.0 -> 5.8 us, 784 x 128 x 1152 6.8 -> 5.7, 49 x 512 x 4608 8.8 -> 8.0; bf16 784 x 512 x
// 128 4.1 -> 2.9, 3136 x 256 x 64 3.8 -> 3.0, 196 x 256 x 1024 3.6 -> 2.8 (with WaveEpilogue's order of loads and stores).
template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {  // f(I), ..., f(N - 1), as compile-time constants
  if constexpr (I < N) {
    f(std::integral_constant<int, I>());
    static_for<I + 1, N>(f);
  }
}
// n chunks through DC slots: load(slot) requests the next chunk into a slot, step(slot, refill) computes the next chunk and, if refill,
// requests the one DC chunks further on into the same slot, begun() is called once when the first chunks are on their way.
// What n leaves over by DC goes behind the loop, with an end for each remainder, or (LEAD) in front of it, through the last slots, so
// that one end serves every n.  LEAD takes fewer registers: fp32 tiles of 16 x 32 117 instead of 150, so that a CU has room for two
// workgroups, 196 x 256 x 2304 on 64 CUs 12.7 -> 11.1 us, ResNet-50's frame of 189 x 253 there 494 -> 482; bf16 tiles of 32 x 64 157 and
// 163 (four waves, two) instead of 188 and 196, three waves on a SIMD instead of two, 900 x 384 x 384 on 64 CUs 5.6 -> 4.7, 4225 x 256 x 288 on 256 5.5 -> 4.8,
// 400 such layers 5.3 % faster.  But nothing may be requested between the first chunks and the loop then, since the paths
// into the loop would differ in what is on its way and the first steps wait for more than they need (begun() comes first);
// the other bf16 tiles have the registers, and their frames are 0.8 % faster with the ends behind the loop.
// AHEAD: begun() comes first for walks without a loop too (bf16 tiles of 32 x 64 with one or two chunks: 2.39 us that way, 2.26).
template <int DC, bool LEAD, bool AHEAD, typename Load, typename Begun, typename Step>
__device__ __forceinline__ void rows_pipeline(const int n, Load&& load, Begun&& begun, Step&& step) {
  auto refilled = [&](auto s) { step(s, std::true_type()); };
  if constexpr (AHEAD) begun();
  if (n < DC) {
    static_for<0, DC>([&](auto k) {
      if (n == k) {
        static_for<0, k>(load);
        if constexpr (!AHEAD) begun();
        static_for<0, k>([&](auto s) { step(s, std::false_type()); });
      }
    });
  } else if constexpr (LEAD) {
    if constexpr (!AHEAD) begun();
    const int lead = n % DC;
    static_for<0, DC>([&](auto r) {
      if (lead == r) {
        static_for<0, DC>([&](auto i) { load(std::integral_constant<int, (DC - r + i) % DC>()); });
        static_for<DC - r, DC>(refilled);
      }
    });
    for (int rounds = n / DC; rounds > 1; --rounds) static_for<0, DC>(refilled);
    static_for<0, DC>([&](auto s) { step(s, std::false_type()); });
  } else {
    static_for<0, DC>(load);
    if constexpr (!AHEAD) begun();
    int left = n - DC;  // chunks still to be requested
    for (; left >= DC; left -= DC) static_for<0, DC>(refilled);
    static_for<0, DC>([&](auto r) {
      if (left == r) {
        static_for<0, r>(refilled);
        static_for<0, DC>([&](auto s) { step(std::integral_constant<int, (r + s) % DC>(), std::false_type()); });
      }
    });
  }
}
// One chunk through the matrix pipe: the two steps (bf16), or the six products of the operands' parts from the smallest to the largest.
template <bool BF16, int R, int TN, int TM = 1>
__device__ __forceinline__ void wave_mma(const Split8 (&a)[TM], const uint4 (&b)[TN][BF16 ? 2 : 3], WaveAcc<R> (&acc)[TM * TN]) {
  constexpr int PA[6] = {BF16 ? 0 : 2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
  for (int t = 0; t < (BF16 ? 2 : 6); ++t)
#pragma unroll
    for (int j = 0; j < TM * TN; ++j) {
      const uint4 l = a[j / TN].p[PA[t]], r = b[j % TN][PB[t]];
      if constexpr (R == 32) acc[j] = mfma_bf16(l, r, acc[j]);
      else acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, l), __builtin_bit_cast(bf16x8, r), acc[j], 0, 0, 0);
    }
}
// LARGE: tensors of 2 GiB and more, whose byte offsets count from what the tile touches instead of from the tensor's start.  (Everywhere,
// it would cost each launch 0.02 to 0.06 us in front of its first load: ResNet-18's frame 133.2 -> 134.5 us.)  Straight into registers
// (gather mode 1), 2250000 x 64 x 256 in fp32 takes 1810 us instead of 1290 on 128 CUs, 2250000 x 64 x 2304 10070 instead of 5540 (with three
// taps per fetch); bf16 with K twice as long 1580 instead of 1120, 8250 instead of 4310.
// POINT: 1 x 1 windows without padding.  There is one tap, which every pixel has, so a lane's rows lie one behind the other, and the walk from tap to tap, some
// fifty instructions for every request, is gone: the first matrix instruction of a wave is the 360th instead of the 620th.  us on 128 CUs without and with: bf16
// 784 x 128 x 512 2.69, 2.45, 196 x 256 x 1024 2.83, 2.65, 49 x 2048 x 512 2.76, 2.56; fp32 784 x 128 x 512 4.09, 3.86, 196 x 64 x 384 2.59, 2.37, 49 x 2048 x 512
// 4.18, 3.95; but bf16 784 x 512 x 128 2.82, 2.86.
template <bool BF16, int R, int TN, int NW, bool LARGE = false, bool POINT = false>
__device__ __forceinline__ void conv_rows_body(const ConvArgs& p, const int mt, const int g, float* const red) {
  constexpr int ES = BF16 ? 2 : 4;
  constexpr int RK = 64 / ES;                     // k of a row
  constexpr int KS = R == 32 ? RK / 2 : RK;       // k of a step
  constexpr int NP = BF16 ? 2 : 3;                // 16-byte pieces of a chunk's weights per lane and channel block: steps, or parts
  // chunks of rows and of weights in flight (bf16 tiles of 32 x 64, 784 x 512 x 128: three 2.9 us, two 3.1; 49 x 512 x 4608 in fp32:
  // 8.3, 8.0; four, in bf16, take so many registers that 3136 x 256 x 64 goes from 3.0 to 4.2)
  constexpr int DC = BF16 && R == 32 && TN == 2 && !POINT ? 3 : 2;  // (POINT: with three the tiles of 32 x 64 have no registers for three waves on a SIMD)
  constexpr int kOutside = (int)0x80000000;       // an offset past the end of any tensor

  if (p.wave_prio) __builtin_amdgcn_s_setprio(3);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: keeps the K loop's control flow scalar
  const int zi = p.splitk == 1 ? 0 : g / p.NTn;
  const int m0 = mt * R, nb0 = (g - zi * p.NTn) * TN;
  const int s_wg0 = zi * p.sz;
  const int s_wg1 = min(s_wg0 + p.sz, p.S);
  const int sbeg = min(s_wg0 + wave * p.sw, s_wg1);
  const int nsteps = min(sbeg + p.sw, s_wg1) - sbeg, nchunks = (nsteps + 1) >> 1;

  // Walk over k = (tap, ci): a row never straddles a tap, so the walk is wave-uniform and lives in scalars.  A lane's row offsets
  // change only from tap to tap; inside one, a scalar offset advances.
  static_assert(!LARGE || !POINT, "one form or the other");
  constexpr int NX = R / 16;  // pixels of a lane
  const int kbeg = sbeg * KS;
  const int tap = POINT ? 0 : fast_div(kbeg, p.mg_cin);
  int ci = kbeg - tap * p.Cin;
  int ky = POINT ? 0 : fast_div(tap, p.mg_kw), kx = tap - ky * p.kw;
  const int piece = lane & 3, prow = lane >> 2;
  int iy0[NX], ix0[NX], rbase[NX], vo[NX];
  const int iy_first = LARGE ? min(max(fast_div(m0, p.mg_wo) * p.stride - p.pad, 0), p.H - 1) : 0;  // the first row of the image that the tile may read
#pragma unroll
  for (int j = 0; j < NX; ++j) {
    const int m = min(m0 + 16 * j + prow, p.M - 1);  // (past the last pixel: the last one once more, whose sums nobody stores)
    if constexpr (POINT) {
      int from = m;
      if (p.stride != 1) {
        const int y = fast_div(m, p.mg_wo);
        from = y * (p.stride * p.W) + (m - y * p.Wo) * p.stride;
      }
      vo[j] = (int)((uint32_t)from * (uint32_t)(p.Cin * ES)) + piece * 16;
      continue;
    }
    const int y = fast_div(m, p.mg_wo), x = m - y * p.Wo;
    iy0[j] = y * p.stride - p.pad;
    ix0[j] = x * p.stride - p.pad;
    rbase[j] = (int)(((uint32_t)(iy0[j] - iy_first) * (uint32_t)p.W + (uint32_t)ix0[j]) * (uint32_t)(p.Cin * ES)) + piece * 16;
  }
  // (LARGE: what lies outside the image is found by its coordinates, so that 2 GiB will do for the size)
  void* from = const_cast<void*>(p.x);
  if constexpr (LARGE) from = (unsigned char*)from + (size_t)(uint32_t)(iy_first * p.W) * (uint32_t)(p.Cin * ES);
  const auto xrsrc = __builtin_amdgcn_make_buffer_rsrc(from, 0, LARGE ? kOutside : (int)((uint32_t)(p.H * p.W) * (uint32_t)p.Cin * ES), 0x00027000);
  int soff = ci * ES, rest = R == 32 ? nchunks : nsteps, left;  // rows of the slice behind this tap's, rows of this tap to go
  auto enter_tap = [&]() {  // at (ky, kx, ci)
    left = min((int)((uint32_t)(p.Cin - ci) / RK), rest);
    rest -= left;
    const int off = (ky * p.W + kx) * p.Cin * ES;
#pragma unroll
    for (int j = 0; j < NX; ++j) {
      const bool in = left > 0 && (unsigned)(iy0[j] + ky) < (unsigned)p.H && (unsigned)(ix0[j] + kx) < (unsigned)p.W;
      vo[j] = in ? rbase[j] + off : kOutside;
    }
  };
  auto next_row = [&]() {
    soff += 64;
    if (--left == 0) {  // wave-uniform; past the slice left is 0 and falls from there, and every row is outside
      ci = soff = 0;
      if (++kx == p.kw) { kx = 0; ++ky; }
      enter_tap();
    }
  };
  if constexpr (!POINT) enter_tap();
  uint4 rows[DC][2];
  auto load_rows = [&](int s) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if constexpr (POINT) {
        const bool past = BF16 && R == 16 && rest <= 0;  // (the second step of a chunk of one)
        rows[s][j] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(xrsrc, past ? kOutside : vo[j % NX], soff, 0));
        if (BF16 && R == 16) --rest;
        if (R == 16 || j == 1) soff += 64;
        continue;
      }
      rows[s][j] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(xrsrc, vo[j % NX], soff, 0));
      if (R == 16 || j == 1) next_row();
    }
  };
  const int wbytes = BF16 ? nsteps * 1024 : nchunks * NP * 1024;
  const unsigned char* const wbase = (const unsigned char*)p.w + ((size_t)nb0 * p.S + sbeg) * (NP * 512);
  __amdgpu_buffer_rsrc_t wrsrc[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) wrsrc[j] = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(wbase) + (size_t)j * p.S * (NP * 512), 0, wbytes, 0x00027000);
  int woff = 0;
  uint4 bw[DC][TN][NP];
  auto load_w = [&](int s) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < NP; ++q) bw[s][j][q] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wrsrc[j], lane * 16 + q * 1024, woff, 0));
    woff += NP * 1024;
  };
  WaveEpilogue<BF16, R, TN, NW, true, LARGE> fin;
  WaveAcc<R> acc[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) acc[j] = WaveAcc<R>(0.f);

  uint4* const st = reinterpret_cast<uint4*>(red) + wave * 128;  // 32 rows of 4 pieces
  const int li = lane % R, lh = lane / R;
  // lanes exchange data through the wave's buffer: order the accesses of the whole wave, not only of each lane
  auto wave_order = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  rows_pipeline<DC, !BF16 || (R == 32 && TN == 2), !BF16>(
      nchunks,
      [&](auto s) {
        load_rows(s);
        load_w(s);
      },
      [&]() { fin.fetch(p, m0, nb0, tid); },
      [&](auto s, auto refill) {
        wave_order();
#pragma unroll
        for (int j = 0; j < 2; ++j) st[(16 * j + prow) * 4 + (piece ^ ((prow >> 1) & 3))] = rows[s][j];  // spread over the banks
        if constexpr (refill) load_rows(s);
        wave_order();
        uint4 a[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          // pieces of the lane's pixel from the chunk's first k on: bf16 R = 32: 2 h + lh, R = 16: 4 h + lh; fp32: 2 lh + h
          const int at = BF16 ? (R == 32 ? 2 : 4) * h + lh : 2 * lh + h;
          a[h] = st[(R == 32 ? li : 16 * (at >> 2) + li) * 4 + ((at & 3) ^ ((li >> 1) & 3))];
        }
        Split8 parts[1];
        if constexpr (BF16) {
          parts[0].p[0] = a[0];
          parts[0].p[1] = a[1];
        } else {
          parts[0] = split8(a[0], a[1]);
        }
        wave_mma<BF16, R, TN>(parts, bw[s], acc);
        __builtin_amdgcn_sched_barrier(0);  // the refill takes over the registers of the slot just used
        if constexpr (refill) load_w(s);
      });
  __syncthreads();  // the partial tiles reuse the LDS of every wave's staging buffer
  fin.template finish<3>(p, DwFusedArgs(), acc, red, m0, nb0, zi, sbeg, nsteps);
}
// ---- the same for 3 x 3 windows with stride 1 and padding 1: one fetch of rows serves three taps (gather mode 5) ---------------
//
// A tile's R pixels and their left and right neighbours are R + 2 consecutive pixels of the input, whatever row of the image they
// lie in.  K is walked as (ky, channels of a chunk, kx): three load instructions bring the rows of three chunks instead of six.  They go
// into 48 places of the wave's corner of LDS (R = 16: the chunk's two rows of a pixel 24 places apart); the places behind them are
// filled with zeros, and there a lane finds its neighbour on the other side of the image's edge.  Above and below the image the
// rows are offsets outside the tensor.  In fp32 the rows are split into their parts on the way into LDS, once for three taps instead of
// for each (split8 is two thirds of a chunk's vector instructions), each part in a plane of its own.  The plan makes every wave's K
// slice a whole number of groups of three chunks; a group's rows and weights are in flight while the one before is computed.  us on 128 CUs without and with: fp32 784 x 128 x 1152 5.85, 5.38
// (split behind LDS 5.48); 196 x 256 x 2304 7.05, 6.67; 49 x 512 x 4608 7.95, 7.25 (7.70); 3136 x 64 x 576 5.88, 5.68 (5.87); 196 x 512 x 4608 13.1, 12.4; bf16 784 x 128 x 1152 3.35, 2.89; 196 x 256 x 2304 4.00,
// 3.57; 49 x 512 x 4608 4.25, 3.64.
// TM = 2 (R = 16): two blocks of pixels (a run of 2 R + 2) and one of channels to a wave, in place of one and two.  A group of three chunks takes 3 load
// instructions for the rows of a block of pixels, 5 for those of two, and 9 (bf16 6) for the weights of a block of channels: 14 (11) for two blocks of
// pixels, 21 (15) for two of channels.  Every sum has the same terms in the same order.  us with two blocks of channels / of pixels: fp32 196 x 256 x 2304 on
// 128 CUs 6.65 / 6.33, 48 x 512 x 4608 on 64 CUs 10.3 / 9.6, bf16 196 x 256 x 2304 3.56 / 3.48.  With R = 32 the loop is shorter and more rows to split in
// front of it cost what fewer loads give: 3136 x 64 x 576 fp32 5.7 / 5.8, bf16 3.1 / 3.3.
// A wave's share of K = steps [s0, s1) where a fetch serves three taps: groups of six steps, `most` at most, each wave that many as long as there are any.
// Waves w and w + 4 run on one SIMD, so that twelve groups on eight waves were four on two SIMDs and two on the others: where that spares a SIMD a group, the
// first waves have `most` and the last ones a group less (fp32 on 128 CUs, 3136 x 64 x 576 5.75 -> 5.25 us; on 64 in 64-pixel tiles 9.9 -> 9.2).  Elsewhere all that more waves
// have is their start: nine groups, three on the busiest SIMD either way, 161 x 64 x 864 on 160 CUs 3.29 -> 3.47.  bf16's four waves have a SIMD each.
template <bool BF16, int NW>
__device__ __forceinline__ void tap_slice(const int s0, const int s1, const int most, const int wave, int* const begin, int* const steps) {
  *begin = min(s0 + wave * most, s1);
  *steps = min(*begin + most, s1) - *begin;
  if constexpr (!BF16 && NW == 8) {
    const int lack = NW * most - (s1 - s0), less = 6 * (wave - NW) + lack;
    if (lack >= 24 && lack <= min(3 * most, 42)) {  // four to seven groups, and the fifth wave would have `most` (a workgroup that has the rest of K split across workgroups may lack more)
      *begin = s0 + wave * most - max(less, 0);
      *steps = most - (less >= 0 ? 6 : 0);
    }
    asm volatile("" : "+s"(*begin), "+s"(*steps));  // (two plain numbers: a K loop for each case takes more registers than there are)
  }
}

template <int TM>
constexpr int conv_taps_places() {  // rows that a wave's corner of LDS holds
  return TM == 1 ? 48 : 80;
}
template <bool BF16, int TM = 1>
constexpr int conv_taps_stage() {  // floats of a wave's corner of LDS
  return BF16 ? conv_taps_places<TM>() * 16 : 3 * conv_taps_places<TM>() * 8;
}
template <bool BF16, int R, int TN, int NW, int TM = 1>
constexpr int conv_taps_lds() {
  return NW * conv_taps_stage<BF16, TM>() > NW * TM * TN * R * R ? NW * conv_taps_stage<BF16, TM>() : NW * TM * TN * R * R;
}
// KEEP as in WaveEpilogue::finish; ahead(): what else is to be on its way while the last group is multiplied.
struct Nothing {
  __device__ __forceinline__ void operator()() const {}
};
template <bool BF16, int R, int TN, int NW, bool LARGE = false, int TM = 1, bool KEEP = false, typename Ahead = Nothing>  // LARGE as in conv_rows_body
__device__ __forceinline__ void conv_taps_body(const ConvArgs& p, const int mt, const int g, float* const red, Ahead&& ahead = Ahead(), unsigned char* const kept = nullptr, const int kept_row = 0) {
  constexpr int ES = BF16 ? 2 : 4;
  constexpr int RK = 64 / ES;                    // k of a row
  constexpr int CK = R == 32 ? RK : 2 * RK;      // k of a chunk, which is two steps
  constexpr int NP = BF16 ? 2 : 3;               // 16-byte pieces of a chunk's weights per lane and channel block: steps, or parts
  constexpr int LOADS = conv_taps_places<TM>() / 16, HALF = conv_taps_places<TM>() / 2;  // HALF: places between a pixel's two rows (R = 16)
  constexpr int kZeros = TM * R + (R == 32 ? 8 : 4);  // a place that holds zeros (R = 16: and the one HALF further on)
  constexpr int kOutside = (int)0x80000000;      // an offset past the end of any tensor

  if (p.wave_prio) __builtin_amdgcn_s_setprio(3);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: keeps the K loop's control flow scalar
  const int zi = p.splitk == 1 ? 0 : g / p.NTn;
  const int m0 = mt * R * TM, nb0 = (g - zi * p.NTn) * TN;
  const int s_wg0 = zi * p.sz;
  const int s_wg1 = min(s_wg0 + p.sz, p.S);
  int sbeg, nsteps;
  tap_slice<BF16, NW>(s_wg0, s_wg1, p.sw, wave, &sbeg, &nsteps);

  const int gk = sbeg / 6 * CK;
  int ky = fast_div(gk, p.mg_cin), ci = gk - ky * p.Cin;
  const int piece = lane & 3, prow = lane >> 2, row_bytes = p.Cin * ES;
  const int base = LARGE ? max(m0 - 1 - p.W, 0) : 0;  // the first pixel that the tile may read
  int first[LOADS];  // byte offset of the lane's piece of its row in each load, at (ky = 0, ci = 0)
  bool used[LOADS];
#pragma unroll
  for (int r = 0; r < LOADS; ++r) {
    const int place = 16 * r + prow, half = R == 16 && place >= HALF ? 1 : 0, row = place - HALF * half;
    used[r] = row < TM * R + 2;
    first[r] = (int)((uint32_t)(m0 - 1 + row - p.W - base) * (uint32_t)row_bytes) + 64 * half + piece * 16;
  }
  void* from = const_cast<void*>(p.x);
  int bytes = p.H * p.W * row_bytes;
  if constexpr (LARGE) {
    from = (unsigned char*)from + (size_t)(uint32_t)base * (uint32_t)row_bytes;
    const uint64_t behind = (uint64_t)(uint32_t)(p.H * p.W - base) * (uint32_t)row_bytes;
    bytes = behind < (uint32_t)kOutside ? (int)behind : kOutside;
  }
  const auto xrsrc = __builtin_amdgcn_make_buffer_rsrc(from, 0, bytes, 0x00027000);
  uint4 rows[LOADS];
  auto load_rows = [&]() {
    const uint32_t off = (uint32_t)(ky * p.W) * (uint32_t)row_bytes + (uint32_t)(ci * ES);
#pragma unroll
    for (int r = 0; r < LOADS; ++r) rows[r] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(xrsrc, used[r] ? (int)((uint32_t)first[r] + off) : kOutside, 0, 0));
    ci += CK;
    if (ci >= p.Cin) {
      ci = 0;
      ++ky;
    }
  };
  const int wbytes = BF16 ? nsteps * 1024 : (nsteps >> 1) * NP * 1024;
  const unsigned char* const wbase = (const unsigned char*)p.w + ((size_t)nb0 * p.S + sbeg) * (NP * 512);
  __amdgpu_buffer_rsrc_t wrsrc[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) wrsrc[j] = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(wbase) + (size_t)j * p.S * (NP * 512), 0, wbytes, 0x00027000);
  int woff = 0;
  uint4 bw[3][TN][NP];
  auto load_w = [&](int kx) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < NP; ++q) bw[kx][j][q] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wrsrc[j], lane * 16 + q * 1024, woff, 0));
    woff += NP * 1024;
  };
  WaveEpilogue<BF16, R, TN, NW, true, LARGE, TM> fin;
  // Bias and residual are requested first: behind the first rows they would leave the paths into the loop with different loads on
  // their way (see rows_pipeline).  fp32 tiles of 16 x 32 keep their registers for the loop (eight waves fit 128, two workgroups a CU:
  // 196 x 256 x 2304 on 64 CUs 10.2 us instead of 12.0) and request them ahead of the last group, which costs the others 0.1 us.
  constexpr bool LATE = !BF16 && R == 16 && TM * TN == 2;
  if constexpr (!LATE) fin.fetch(p, m0, nb0, tid);
  WaveAcc<R> acc[TM * TN];
#pragma unroll
  for (int j = 0; j < TM * TN; ++j) acc[j] = WaveAcc<R>(0.f);

  // bf16: places of 4 pieces of 16 bytes; fp32: in each of three planes places of 16 values in bf16, 2 pieces of 16 bytes
  uint4* const st = reinterpret_cast<uint4*>(red) + wave * (conv_taps_stage<BF16, TM>() / 4);
  constexpr int PLANE = conv_taps_places<TM>() * 2;
  const int li = lane % R, lh = lane / R;
  // Pieces of the lane's pixel from the chunk's first k on: bf16 R = 32: 2 h + lh, R = 16: 4 h + lh (h = 0, 1); fp32: 8 k from 8 lh on.
  // row_at: where piece h = 0 of a row lies, or its part in the first plane (spread over the banks)
  auto row_at = [&](int row) {
    const int place = row + (R == 16 && !BF16 ? HALF * (lh >> 1) : 0);
    return BF16 ? place * 4 + (lh ^ ((place >> 1) & 3)) : place * 2 + ((lh & 1) ^ ((place >> 2) & 1));
  };
  const int m = m0 + li, x = m - fast_div(m, p.mg_wo) * p.Wo;
  int at[TM][3] = {{x == 0 ? row_at(kZeros) : row_at(li), row_at(li + 1), x == p.Wo - 1 ? row_at(kZeros) : row_at(li + 2)}};
  if constexpr (TM == 2) {
    const int x2 = m + R - fast_div(m + R, p.mg_wo) * p.Wo;
    at[TM - 1][0] = x2 == 0 ? row_at(kZeros) : row_at(R + li);
    at[TM - 1][1] = row_at(R + li + 1);
    at[TM - 1][2] = x2 == p.Wo - 1 ? row_at(kZeros) : row_at(R + li + 2);
  }
  // lanes exchange data through the wave's buffer: order the accesses of the whole wave, not only of each lane
  auto wave_order = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  auto chunk = [&](auto kx, auto more) {  // tap kx of a group; more: another group follows
    if constexpr (kx == 0) {
      wave_order();
#pragma unroll
      for (int r = 0; r < LOADS; ++r) {
        if constexpr (BF16) {
          st[(16 * r + prow) * 4 + (piece ^ ((prow >> 1) & 3))] = rows[r];
        } else {
          const Split4 v = split4(rows[r]);
#pragma unroll
          for (int q = 0; q < 3; ++q) reinterpret_cast<uint2*>(st + q * PLANE + (16 * r + prow) * 2 + ((piece >> 1) ^ ((prow >> 2) & 1)))[piece & 1] = v.p[q];
        }
      }
      if constexpr (more) load_rows();
      wave_order();
    }
    Split8 parts[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if constexpr (BF16) {
        parts[i].p[0] = st[at[i][kx]];
        parts[i].p[1] = st[R == 32 ? at[i][kx] ^ 2 : at[i][kx] + 4 * HALF];
      } else {
#pragma unroll
        for (int q = 0; q < 3; ++q) parts[i].p[q] = st[q * PLANE + at[i][kx]];
      }
    }
    wave_mma<BF16, R, TN, TM>(parts, bw[kx], acc);
    __builtin_amdgcn_sched_barrier(0);  // the refill takes over the registers of the weights just used
    if constexpr (more) load_w(kx);
  };
  if (nsteps > 0) {
    load_rows();
    static_for<0, 3>(load_w);
    // (A pixel past the output is a pixel of zeros: see drop_pixels.  25 x 512 x 4608 with K split over 240 CUs: 7.05 us with the neighbours' sums,
    // 7.22 with sums dropped, 7.10 so.)
    if (!BF16 && __builtin_expect(m0 + TM * R > p.M, 0)) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k) at[i][k] = m + R * i < p.M ? at[i][k] : row_at(kZeros);
    }
    for (int groups = nsteps / 6; groups > 1; --groups) static_for<0, 3>([&](auto kx) { chunk(kx, std::true_type()); });
    if constexpr (LATE) fin.fetch(p, m0, nb0, tid);
    if constexpr (!KEEP) static_for<0, 3>([&](auto kx) { chunk(kx, std::false_type()); });
  } else if constexpr (LATE) {
    fin.fetch(p, m0, nb0, tid);
  }
  if constexpr (KEEP) {  // (in both branches above, its loads would count as on their way in the other one as well, and every wait would be for all)
    ahead();
    if (nsteps > 0) static_for<0, 3>([&](auto kx) { chunk(kx, std::false_type()); });
  }
  __syncthreads();  // the partial tiles reuse the LDS of every wave's staging buffer
  fin.template finish<5, KEEP>(p, DwFusedArgs(), acc, red, m0, nb0, zi, sbeg, nsteps, kept, kept_row);
}

template <int R, int TN, int NW>
constexpr int conv_rows_lds() {  // floats of LDS
  return NW * 512 > NW * TN * R * R ? NW * 512 : NW * TN * R * R;
}

// ---- the network input in patches (gather mode 6) ---------------------------------------------------------------------------
//
// An input of up to four channels leaves a lane nothing to load but single values, eight plane loads a chunk of 16 k, and every input
// pixel is wanted by k * k / stride^2 taps: the vector memory unit, twenty cycles for every load instruction of a CU, bounds the gather
// of conv_wave_body.  Here a workgroup of four waves fetches the input pixels of its tile once, a load a plane, splits them into their
// parts (bf16: rounds them) and keeps them in LDS as pixels of four channels, 8 bytes a part; the zeros outside the image come from
// the buffer descriptor.  A lane reads a tap with one instruction a part, one chunk ahead of the matrix pipe.  The columns of a row lie
// by their remainder by the stride, so that neighbouring output pixels read neighbouring places whatever the stride.  Where a tap lies is
// looked up in a table that the workgroup makes while its pixels are on their way (the same in scalars, tap by tap, took as long as
// the products).  K is not split: WN waves side by side own 32 channels each, 4 / WN below one another two rows of 16 pixels each, and
// each walks all of K, in the order (tap, channel) of the packed weights, with DC chunks of weights in flight; taps past the last one
// are a place of zeros.  Two blocks of pixels to a wave (a weight serves both) need so many registers that fewer workgroups hide
// each other's waits: 6.1 us, 4.6, 6.0, 8.7 in place of the following.  us on 128 CUs, gather -> patches: 12544 x 64 x 7 x 7 with stride 2 fp32
// 10.3 -> 5.8 (192 CUs 10.0 -> 5.7, 64 CUs 16.4 -> 8.4), bf16 7.2 -> 4.3; 50176 x 64 x 3 x 3 10.7 -> 6.4; 12544 x 32 x 3 x 3 with stride 2 3.5 -> 3.2;
// 1024 x 16 x 3 x 3 3.05 -> 2.8.
// POOL: the 3 x 3 max pooling with stride 2 and padding 1 behind the convolution in the same launch, for two channel blocks side by side.  A workgroup of
// ten waves computes ten rows of 16 outputs, of which nine rows of 15 are the windows of 4 x 7 pooled pixels, and passes them through LDS; they
// are never stored.  1.4 outputs are computed for one that counts, in place of a launch.
template <bool BF16, bool POOL>
constexpr int conv_image_lds() {  // floats of LDS
  constexpr int kPatch = (BF16 ? 1 : 3) * ((POOL ? kImagePoolPatch : kImagePatch) + 1) * 2 + kImageTaps, kTiles = (POOL ? 2 * kImagePoolRows + 2 : 4) * 1024;
  return kPatch > kTiles ? kPatch : kTiles;
}
template <bool BF16, int WN, bool POOL>
__device__ __forceinline__ void conv_image_body(const ImageConvArgs& p, const int L, float* const lds) {
  static_assert(!POOL || WN == 2, "pooled tiles are two channel blocks wide");
  constexpr int ES = BF16 ? 2 : 4, NP = BF16 ? 1 : 3, DC = BF16 ? 4 : 2, NT = POOL ? 128 * (kImagePoolRows + 1) : 256;
  constexpr int PATCH = POOL ? kImagePoolPatch : kImagePatch, PLANE = PATCH + 1, ROUNDS = (PATCH + NT - 1) / NT;
  constexpr int kOutside = (int)0x80000000;  // an offset past the end of any tensor
  if (p.wave_prio) __builtin_amdgcn_s_setprio(3);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 31, lh = lane >> 5;
  const int g = fast_div(L, p.mg_tiles), tile = L - g * p.tiles;
  const int ty = fast_div(tile, p.mg_across), tx = tile - ty * p.across;
  const int x0 = POOL ? tx * 2 * kImagePoolCols - 1 : tx * kImageCols, y0 = POOL ? ty * 2 * kImagePoolRows - 1 : ty * (8 / WN);  // (POOL: from -1 on)
  const int nb = g * WN + wave % WN, row0 = wave / WN * 2;  // the wave's channel block and its first row of the tile

  const int plane = p.H * p.W * 4;
  const auto irsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.x), 0, p.c_real * plane, 0x00027000);
  const int po1 = min(1, p.c_real - 1) * plane, po2 = min(2, p.c_real - 1) * plane;
  auto by_stride = [&](int x) {  // (a select; a branch of its own for strides of one costs more)
    const int q = (int)__umulhi((uint32_t)x, p.mg_stride);
    return p.stride == 1 ? x : q;
  };
  uint4 px[ROUNDS];
  int place[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    place[r] = 0;
    px[r] = make_uint4(0u, 0u, 0u, 0u);
    if (NT * r < p.patch) {
      const int i = tid + NT * r, y = (int)__umulhi((uint32_t)i, p.mg_patch_w), x = i - y * p.patch_w, iy = y0 * p.stride - p.pad + y, ix = x0 * p.stride - p.pad + x;
      const int col = by_stride(x);
      place[r] = y * p.pitch + (x - col * p.stride) * p.phase + col;
      const int o = i < p.patch && (unsigned)iy < (unsigned)p.H && (unsigned)ix < (unsigned)p.W ? (iy * p.W + ix) * 4 : kOutside;
      px[r].x = __builtin_amdgcn_raw_buffer_load_b32(irsrc, o, 0, 0);
      px[r].y = __builtin_amdgcn_raw_buffer_load_b32(irsrc, o, po1, 0);  // (planes past the last one repeat it; their weights are zero)
      px[r].z = __builtin_amdgcn_raw_buffer_load_b32(irsrc, o, po2, 0);
      if (p.c_real > 3) px[r].w = __builtin_amdgcn_raw_buffer_load_b32(irsrc, o, 3 * plane, 0);
    }
  }
  const int n = POOL ? g * 64 + 4 * (tid & 15) : nb * 32 + 4 * lane % 32;  // first channel of the lane's quads
  const auto brsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.bias), 0, p.Cout * 4, 0x00027000);
  const float4 bias = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(brsrc, n * 4, 0, 0));

  const int chunks = BF16 ? p.S : p.S >> 1;  // of 16 k
  const auto wrsrc = __builtin_amdgcn_make_buffer_rsrc((unsigned char*)const_cast<void*>(p.w) + (size_t)nb * chunks * (NP * 1024), 0, chunks * (NP * 1024), 0x00027000);
  int woff = 0;
  uint4 bw[DC][NP];
  auto load = [&](int s) {
#pragma unroll
    for (int q = 0; q < NP; ++q) bw[s][q] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, lane * 16 + q * 1024, woff, 0));
    woff += NP * 1024;
  };

  uint2* const st = reinterpret_cast<uint2*>(lds);
  int base = (row0 + li / 16) * p.stride * p.pitch + li % 16;  // place of the lane's pixel under the first tap
  const int* const taps = reinterpret_cast<const int*>(lds + NP * PLANE * 2) + (BF16 ? lh : 2 * lh);
  int tap = 0;
  int2 o = make_int2(0, 0);  // places of the next chunk's taps
  auto read_taps = [&]() {
    if constexpr (BF16) o.x = taps[tap];
    else o = *(const int2*)(taps + tap);
    tap += BF16 ? 2 : 4;
  };
  uint4 next[NP];  // the next chunk's pixels
  auto read = [&]() {
    const int at = min(base + o.x, PATCH), bt = min(base + o.y, PATCH);
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const uint2 u = st[q * PLANE + at], v = BF16 ? make_uint2(0u, 0u) : st[q * PLANE + bt];  // (bf16: eight k are one tap, the upper four zero)
      next[q] = make_uint4(u.x, u.y, v.x, v.y);
    }
    read_taps();
  };
  f32x16 acc[1] = {f32x16(0.f)};
  // All slots are filled before the patch is waited for (weights past the last chunk are zeros, and so are its taps), what the chunks
  // leave over by DC goes through the last slots first, so that there is one end.
  const int n_chunks = max(chunks, DC), lead = n_chunks % DC;
  static_for<0, DC>([&](auto r) {
    if (lead == r) static_for<0, DC>([&](auto i) { load((DC - r + i) % DC); });
  });
  if (tid < NP) st[tid * PLANE + PATCH] = make_uint2(0u, 0u);
#pragma unroll
  for (int t = tid; t < kImageTaps; t += NT) {
    const int ky = fast_div(t, p.mg_k), kx = t - ky * p.k, col = by_stride(kx);
    reinterpret_cast<int*>(lds + NP * PLANE * 2)[t] = ky < p.k ? ky * p.pitch + (kx - col * p.stride) * p.phase + col : PATCH;
  }
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    if (tid + NT * r < p.patch) {
      if constexpr (BF16) {
        st[place[r]] = make_uint2(pack_bf16_rne(__uint_as_float(px[r].x), __uint_as_float(px[r].y)), pack_bf16_rne(__uint_as_float(px[r].z), __uint_as_float(px[r].w)));
      } else {
        const Split4 v = split4(px[r]);
#pragma unroll
        for (int q = 0; q < NP; ++q) st[q * PLANE + place[r]] = v.p[q];
      }
    }
  }
  // (A pixel past the output is a pixel of zeros: see drop_pixels.  Here that is the cheaper way: first convolutions of few tiles take 0.07 us longer
  // for it and 0.14 for dropped sums.)
  if (!BF16 && (y0 + row0 + 2 > p.Ho || x0 + kImageCols > p.Wo || (POOL && (y0 < 0 || x0 < 0))))
    base = (unsigned)(y0 + row0 + li / 16) < (unsigned)p.Ho && (unsigned)(x0 + li % 16) < (unsigned)p.Wo ? base : PATCH;
  __syncthreads();
  read_taps();
  read();
  auto step = [&](auto s, auto refill) {
    uint4 pixels[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) pixels[q] = next[q];
    read();
    constexpr int PA[6] = {BF16 ? 0 : 2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
    for (int t = 0; t < (BF16 ? 1 : 6); ++t) acc[0] = mfma_bf16(pixels[PA[t]], bw[s][PB[t]], acc[0]);
    __builtin_amdgcn_sched_barrier(0);  // the refill takes over the registers of the weights just used
    if constexpr (refill) load(s);
  };
  auto refilled = [&](auto s) { step(s, std::true_type()); };
  static_for<0, DC>([&](auto r) {
    if (lead == r) static_for<DC - r, DC>(refilled);
  });
  for (int rounds = n_chunks / DC; rounds > 1; --rounds) static_for<0, DC>(refilled);
  static_for<0, DC>([&](auto s) { step(s, std::false_type()); });
  if constexpr (!BF16) {
    if (out_of_range(acc)) {
      const bool small = all_small(acc);
      const f32x16 first = acc[0];
      ConvArgs c = ConvArgs();
      c.x = p.x; c.w = p.w; c.H = p.H; c.W = p.W; c.Cin = 4; c.Wo = p.Wo; c.kh = c.kw = p.k; c.stride = p.stride; c.pad = p.pad;
      c.M = p.M; c.S = p.S; c.mg_wo = p.mg_wo; c.mg_kw = p.mg_k; c.c_real = p.c_real;
      if constexpr (POOL) {  // pixels are counted from -1 on in both directions: an output one row and one column larger, and as much more padding
        c.Wo = p.Wo + 1;
        c.pad = p.pad + p.stride;
        c.M = (p.Ho + 1) * c.Wo;
        c.mg_wo = 0xffffffffu / (uint32_t)c.Wo + 1u;
        plain_products<6, 32, 1, 1>(c, DwFusedArgs(), (y0 + 1 + row0) * c.Wo + x0 + 1, nb, 0, p.S, acc);
      } else {
        plain_products<6, 32, 1, 1>(c, DwFusedArgs(), (y0 + row0) * p.Wo + x0, nb, 0, p.S, acc);
      }
      take_second(small, first, acc[0]);
    }
  }
  __syncthreads();  // the tiles go through the patch's LDS, each wave's through its own corner
  float* const out = lds + wave * 1024;
  if constexpr (POOL) {
#pragma unroll
    for (int v = 0; v < 16; ++v) out[64 * v + lane] = acc[0][v];
    __syncthreads();
    // A thread has four channels of a pooled pixel.  The largest sum is taken before bias and activation, which change no order (NaN never wins).
    const int quad = tid & 15, pp = tid >> 4, py = pp / kImagePoolCols, px2 = 2 * (pp - py * kImagePoolCols);
    const int oy = ty * kImagePoolRows + py, ox = tx * kImagePoolCols + (px2 >> 1);
    if (pp >= kImagePoolRows * kImagePoolCols || oy >= p.pool_h || ox >= p.pool_w) return;
    float best[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
    for (int ky = 0; ky < 3; ++ky)
#pragma unroll
      for (int kx = 0; kx < 3; ++kx) {
        const int r = 2 * py + ky, pixel = r % 2 * 16 + px2 + kx;
        const float4 v = *(const float4*)&lds[(r / 2 * 2 + (quad >> 3)) * 1024 + ((pixel >> 3) * 4 + (pixel & 3)) * 64 + (pixel >> 2 & 1) * 32 + 4 * (quad & 7)];
        const bool in = (unsigned)(y0 + r) < (unsigned)p.Ho && (unsigned)(x0 + px2 + kx) < (unsigned)p.Wo;
        best[0] = in ? fmaxf(best[0], v.x) : best[0]; best[1] = in ? fmaxf(best[1], v.y) : best[1];
        best[2] = in ? fmaxf(best[2], v.z) : best[2]; best[3] = in ? fmaxf(best[3], v.w) : best[3];
      }
    if (n >= p.Cout) return;
    best[0] += bias.x; best[1] += bias.y; best[2] += bias.z; best[3] += bias.w;
    apply_act(best, p.act);
    unsigned char* const to = (unsigned char*)p.y + ((size_t)(oy * p.pool_w + ox) * p.Cout + n) * ES;
    if constexpr (BF16) put(to, make_uint2(pack_bf16_rne(best[0], best[1]), pack_bf16_rne(best[2], best[3])));
    else put(to, make_float4(best[0], best[1], best[2], best[3]));
    return;
  }
  const auto yrsrc = __builtin_amdgcn_make_buffer_rsrc(p.y, 0, p.M * p.Cout * ES, 0x00027000);
#pragma unroll
  for (int v = 0; v < 16; ++v) out[64 * v + lane] = acc[0][v];
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  float val[16];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float4 v = *(const float4*)&out[4 * lane + 256 * r];
    val[4 * r] = v.x + bias.x; val[4 * r + 1] = v.y + bias.y; val[4 * r + 2] = v.z + bias.z; val[4 * r + 3] = v.w + bias.w;
  }
  apply_act(val, p.act);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int pixel = 8 * r + (lane >> 3 & 1) * 4 + (lane >> 4);  // of the block (as in WaveEpilogue)
    const int y = y0 + row0 + pixel / 16, x = x0 + pixel % 16;
    const int at = y < p.Ho && x < p.Wo && n < p.Cout ? ((y * p.Wo + x) * p.Cout + n) * ES : kOutside;
    const float* const v = val + 4 * r;
    if constexpr (BF16) put_at(yrsrc, at, make_uint2(pack_bf16_rne(v[0], v[1]), pack_bf16_rne(v[2], v[3])));
    else put_at(yrsrc, at, make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])));
  }
}

// ---- a 1x1 convolution and the 3x3 depthwise convolution behind it --------------------------------------------------------------
//
// A depthwise channel reads only its own channel of the layer in front, so a workgroup that owns 16 channels of a band of output rows computes those
// channels of the convolution for the rows that the band reads (neighbouring bands compute the rows between them twice), leaves them in LDS, and
// convolves them there: one launch, and the widest tensor of an inverted residual block is never stored.  K is short, NCH chunks of 32 k, so that a wave
// has all pixels and weights of its 16-pixel tile on their way at once; the 16 bytes that lanes load straight into registers are whole cache lines.
// The sums have the order that the convolution by itself has with two waves: the first chunks and the others in accumulators of their own.
// Bound by its chain of waits (arguments, pixels and weights, LDS, stores), behind which two launches have as much again.  us of the two launches / of one, fp32
// on 128 CUs: 784 x 192 x 32 5.4 / 4.0, 196 x 384 x 64 4.5 / 3.85, 196 x 576 x 96 5.0 / 4.7, 49 x 960 x 160 5.0 / 4.2.  Two tiles to a wave (fewer loads of
// weights, twice as long a chain) 3.95, 4.0, 5.1 and 4.85; bands of half as many rows 4.2, 4.1, 4.9 and 4.65, of twice as many 5.4, 4.4, 7.3 and 4.65.
template <bool BF16, int NCH>
__device__ __forceinline__ void conv_expand_dw_body(const ExpandDwArgs& p, const int L, float* const lds) {
  constexpr int ES = BF16 ? 2 : 4, NP = BF16 ? 1 : 3, NA = BF16 ? 1 : 2;
  constexpr int FIRST = (NCH + 1) / 2;    // chunks of the first accumulator
  constexpr int ROW = kExpandRow;
  constexpr int kOutside = (int)0x80000000;
  float* const taps = lds + kExpandPixels * ROW;  // [9][16] weights and [16] biases of the depthwise layer
  if (p.wave_prio) __builtin_amdgcn_s_setprio(3);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lq = lane >> 4;
  const int g = fast_div(L, p.mg_bands), oy0 = (L - g * p.bands) * p.band, oy1 = min(oy0 + p.band, p.Ho);
  const int y0 = max(oy0 * p.stride - 1, 0), y1 = min((oy1 - 1) * p.stride + 1, p.H - 1);  // rows of the convolution
  const int first = y0 * p.W, pixels = (y1 - y0 + 1) * p.W, tiles = (pixels + 15) >> 4;

  const auto xrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.x), 0, p.H * p.W * p.Cin * ES, 0x00027000);
  uint4 a[NCH][NA];
  auto load_pixels = [&](const int t) {  // lane (i, q): pixel i of tile t, k = 8 q .. 8 q + 7 of each chunk
    const int i = 16 * t + li;
    const int at = i < pixels ? (first + i) * p.Cin * ES + lq * 8 * ES : kOutside;  // (a pixel past the band's is a pixel of zeros: see drop_pixels)
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
      for (int h = 0; h < NA; ++h) a[c][h] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(xrsrc, at, c * 32 * ES + h * 16, 0));
  };
  load_pixels(wave);
  const unsigned char* const wb = (const unsigned char*)p.w + (size_t)g * (NCH * NP * 1024) + lane * 16;
  uint4 b[NCH][NP];
#pragma unroll
  for (int c = 0; c < NCH; ++c)
#pragma unroll
    for (int q = 0; q < NP; ++q) b[c][q] = *(const uint4*)(wb + (c * NP + q) * 1024);
  const float bias = p.bias[g * 16 + li];
  const int at_taps = (tid >> 2) * p.C + g * 16 + 4 * (tid & 3);  // (of the first 36 threads; the next four have the biases)
  float4 tap = make_float4(0.f, 0.f, 0.f, 0.f);
  if (tid < 36) {
    if constexpr (BF16) {
      const uint2 u = *(const uint2*)((const uint16_t*)p.dw_w + at_taps);
      tap = make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xffff0000u));
    } else {
      tap = *(const float4*)((const float*)p.dw_w + at_taps);
    }
  } else if (tid < 40) {
    tap = *(const float4*)(p.dw_bias + g * 16 + 4 * (tid & 3));
  }

  auto keep = [&](const int t, const f32x4& sum) {  // outputs of tile t of the convolution
    float v[4] = {sum[0] + bias, sum[1] + bias, sum[2] + bias, sum[3] + bias};
    apply_act(v, p.act);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * t + 4 * lq + r;
      if (i < pixels) lds[i * ROW + li] = BF16 ? bf16_bits_to_f32(f32_to_bf16_bits(v[r])) : v[r];
    }
  };
  for (int t = wave; t < tiles; t += p.threads >> 6) {
    if (t != wave) load_pixels(t);
    f32x4 acc[2][1] = {{f32x4(0.f)}, {f32x4(0.f)}};
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      Split8 parts;
      if constexpr (BF16) parts.p[0] = a[c][0];
      else parts = split8(a[c][0], a[c][NA - 1]);
      constexpr int PA[6] = {BF16 ? 0 : 2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};
      f32x4& s = acc[c >= FIRST][0];
#pragma unroll
      for (int k = 0; k < (BF16 ? 1 : 6); ++k)
        s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, parts.p[PA[k]]), __builtin_bit_cast(bf16x8, b[c][PB[k]]), s, 0, 0, 0);
    }
    if constexpr (!BF16) {
      if (__builtin_expect(out_of_range(acc[0]) || (NCH > 1 && out_of_range(acc[1])), 0)) {
        ConvArgs c = ConvArgs();
        c.x = p.x; c.w = p.w; c.H = p.H; c.W = c.Wo = p.W; c.Cin = p.Cin; c.kh = c.kw = c.stride = 1; c.M = p.H * p.W; c.S = p.S; c.mg_wo = p.mg_w;
        c.mg_cin = 1;  // (every k is below Cin)
#pragma unroll 1
        for (int h = 0; h < 2; ++h) {
          f32x4 s[1];
          plain_products<3, 16, 1, 1>(c, DwFusedArgs(), first + 16 * t, g, h * 2 * FIRST, h ? 2 * (NCH - FIRST) : 2 * FIRST, s);
          const f32x4 had = h ? acc[1][0] : acc[0][0];
          take_second(all_small(had), had, s[0]);
          if (h) acc[1][0] = s[0];
          else acc[0][0] = s[0];
        }
      }
    }
    keep(t, acc[0][0] + acc[1][0]);
  }
  if (tid < 40) *(float4*)&taps[4 * tid] = tap;
  __syncthreads();

  const int items = (oy1 - oy0) * p.Wo * 4;  // a thread has four channels of an output pixel
  for (int it = tid; it < items; it += p.threads) {
    const int quad = it & 3, m = it >> 2, r = fast_div(m, p.mg_wo), ox = m - r * p.Wo, oy = oy0 + r;
    const int iy0 = oy * p.stride - 1, ix0 = ox * p.stride - 1;
    const float4 s = *(const float4*)&taps[144 + 4 * quad];
    float v[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
    for (int t = 0; t < 9; ++t) {  // (the order of dwconv_point)
      const int iy = iy0 + t / 3, ix = ix0 + t % 3;
      const bool in = (unsigned)iy < (unsigned)p.H && (unsigned)ix < (unsigned)p.W;
      const float4 e = *(const float4*)&lds[(in ? (iy - y0) * p.W + ix : 0) * ROW + 4 * quad], w = *(const float4*)&taps[16 * t + 4 * quad];
      v[0] = in ? fmaf(e.x, w.x, v[0]) : v[0]; v[1] = in ? fmaf(e.y, w.y, v[1]) : v[1];
      v[2] = in ? fmaf(e.z, w.z, v[2]) : v[2]; v[3] = in ? fmaf(e.w, w.w, v[3]) : v[3];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = apply_act(v[i], p.dw_act);
    unsigned char* const to = (unsigned char*)p.y + ((size_t)(oy * p.Wo + ox) * p.C + g * 16 + 4 * quad) * ES;
    if constexpr (BF16) put(to, make_uint2(pack_bf16_rne(v[0], v[1]), pack_bf16_rne(v[2], v[3])));
    else put(to, make_float4(v[0], v[1], v[2], v[3]));
  }
}

// ---- the 3x3 convolution of a bottleneck, the 1x1 behind it and the next block's 1x1 -----------------------------------------
//
// Both 1x1 convolutions need nothing but the pixels of the tile, so the workgroup that owns a tile of the 3x3 convolution (32 pixels, all of its 64
// channels: conv_taps_body) leaves it in LDS and goes on: the first 1x1 (kChainWide channels) takes its residual, is stored and stays in LDS, and
// the second (up to 64 channels) reads it there.  Bound by the launch and its chain of waits like the launches that it takes the place of; the weights and
// the residual of each are requested before the one in front is finished, so that nothing of them is waited for.  us of the launches by themselves / of one, 3136 pixels on
// 128 CUs: bf16 with both 1x1 8.7 / 5.6, with the first 6.0 / 5.0; fp32 14.0 / 10.4 and 10.0 / 9.0.  ResNet-50's first group, five launches fewer: frame in bf16
// 202.2 -> 193.1, six tasks saturated 7243 -> 7003, the mixed set (fp32) 10410 -> 10117.
// The sums have the order that launches of their own have: of the first 1x1 two halves of K, each in an accumulator, of the second as many slices as
// waves.  The first has weights and pixels in each other's place in the matrix instruction: a lane then holds four channels in a row of its pixel.
template <bool BF16, int NW>
constexpr int conv_chain_lds() {  // floats of LDS
  return conv_taps_lds<BF16, 32, 2, NW>() + 32 * (64 * (BF16 ? 2 : 4) + 16) / 4 + kChainWide;
}
template <bool BF16, int NW>
__device__ __forceinline__ void conv_chain_body(const ConvArgs& p, const ChainArgs& c, const int mt, float* const lds) {
  constexpr int ES = BF16 ? 2 : 4, NT = NW * 64, NP = BF16 ? 1 : 3;
  constexpr int UNITS = 4, HALF = UNITS / 2;            // 16 k each of the first 1x1
  constexpr int NB = kChainWide / 32 / NW;              // its channel blocks of a wave
  constexpr int S1 = kChainWide / 16, U1 = S1 / NW;     // 16 k each of the second, of a wave's slice of it
  constexpr int ROW = 64 * ES + 16, WIDE = kChainWide * ES + 16;  // bytes of a pixel in LDS, spread over the banks
  constexpr int ROW_VECS = kChainWide * ES / 16;        // 16-byte vectors of a pixel of the wide tile
  constexpr int NV = 32 * ROW_VECS / NT;                // ... of the tile to a thread
  static_assert(32 * WIDE <= conv_taps_lds<BF16, 32, 2, NW>() * 4, "the wide tile lies where the partial tiles were");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 31, lh = lane >> 5, m0 = mt * 32;
  using ResVec = typename std::conditional<BF16, uint2, uint4>::type;
  unsigned char* const kept = (unsigned char*)(lds + conv_taps_lds<BF16, 32, 2, NW>());  // [32][ROW]
  unsigned char* const wide = (unsigned char*)lds;                                       // [32][WIDE]
  float* const biases = lds + conv_taps_lds<BF16, 32, 2, NW>() + 32 * ROW / 4;

  const int u0 = wave * U1;
  uint4 w3[NB][UNITS][NP], w1[U1][2][NP], res[NV];
  float4 bias3;
  const int at0 = mt * (32 * kChainWide * ES);  // a tile's rows lie one behind the other
  WaveEpilogue<BF16, 32, 2, NW, true> fin;
  ConvArgs q = ConvArgs();  // the second 1x1 as the epilogue wants it
  q.bias = c.bias1; q.y = c.y1; q.Cout = c.n1; q.M = p.M; q.act = c.act1; q.splitk = 1;
  auto ahead = [&]() {
    const auto w3rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(c.w3), 0, kChainWide / 32 * UNITS * NP * 1024, 0x00027000);
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int u = 0; u < UNITS * NP; ++u) w3[b][u / NP][u % NP] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(w3rsrc, lane * 16 + u * 1024, (wave + b * NW) * (UNITS * NP * 1024), 0));
    const auto rrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(c.res3), 0, c.res3 ? p.M * (kChainWide * ES) : 0, 0x00027000);  // (past the end, and without a residual: zeros)
#pragma unroll
    for (int r = 0; r < NV; ++r) res[r] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rrsrc, at0 + (tid + r * NT) * 16, 0, 0));
    const auto brsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(c.bias3), 0, kChainWide * 4, 0x00027000);
    bias3 = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(brsrc, tid * 16, 0, 0));  // (of the threads past the last channel: zeros)
  };
  conv_taps_body<BF16, 32, 2, NW, false, 1, true>(p, mt, 0, lds, ahead, kept, ROW);
  {
    const auto w1rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(c.w1), 0, c.n1 ? 2 * S1 * NP * 1024 : 0, 0x00027000);
#pragma unroll
    for (int u = 0; u < U1; ++u)
#pragma unroll
      for (int k = 0; k < 2 * NP; ++k) w1[u][k / NP][k % NP] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(w1rsrc, lane * 16 + ((k / NP * S1 + u0 + u) * NP + k % NP) * 1024, 0, 0));
    fin.fetch(q, m0, 0, tid);
  }
  if (tid < kChainWide / 4) *(float4*)&biases[4 * tid] = bias3;
  __syncthreads();

  auto pixels_of = [&](const unsigned char* const row, const int u) {  // the lane's pixel, k = 16 u + 8 lh .. + 7
    Split8 s;
    if constexpr (BF16) s.p[0] = *(const uint4*)(row + (16 * u + 8 * lh) * ES);
    else s = split8(*(const uint4*)(row + (16 * u + 8 * lh) * ES), *(const uint4*)(row + (16 * u + 8 * lh) * ES + 16));
    return s;
  };
  constexpr int PA[6] = {BF16 ? 0 : 2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};  // (as wave_mma)
#pragma unroll
  for (int r = 0; r < NV; ++r) {
    const int v = tid + r * NT;
    *(uint4*)(wide + v / ROW_VECS * WIDE + v % ROW_VECS * 16) = res[r];
  }
  f32x16 sum[NB];
  {
    f32x16 acc[NB][2];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b][0] = acc[b][1] = f32x16(0.f);
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
      const Split8 a = pixels_of(kept + li * ROW, u);
#pragma unroll
      for (int k = 0; k < (BF16 ? 1 : 6); ++k)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[b][u / HALF] = mfma_bf16(w3[b][u][PB[k]], a.p[PA[k]], acc[b][u / HALF]);
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      if constexpr (!BF16) {
        if (__builtin_expect(out_of_range(acc[b]), 0)) {  // the wave's block once more, on the fp32 matrix instructions
          const f32x16 had[2] = {acc[b][0], acc[b][1]};
#pragma unroll
          for (int h = 0; h < 2; ++h) acc[b][h] = f32x16(0.f);
#pragma unroll
          for (int u = 0; u < UNITS; ++u) {
            float w[3][8];
#pragma unroll
            for (int k = 0; k < 3; ++k) unpack<true>(w3[b][u][k], w[k]);
            const float* const x = (const float*)(kept + li * ROW) + 16 * u + 8 * lh;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[b][u / HALF] = __builtin_amdgcn_mfma_f32_32x32x2f32((w[2][e] + w[1][e]) + w[0][e], x[e], acc[b][u / HALF], 0, 0, 0);
          }
#pragma unroll
          for (int h = 0; h < 2; ++h) take_second(all_small(had[h]), had[h], acc[b][h]);
        }
      }
      sum[b] = acc[b][0] + acc[b][1];
    }
  }
  __syncthreads();  // the residual lies in `wide`: a lane adds its sums and leaves the outputs in its place
  const bool inside = m0 + li < p.M;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    unsigned char* const at = wide + li * WIDE + ((wave + b * NW) * 32 + 4 * lh) * ES;  // four quads of channels, eight channels apart
    const float* const bi = biases + (wave + b * NW) * 32 + 4 * lh;
    float v[16];
    ResVec old[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) old[k] = *(const ResVec*)(at + 8 * k * ES);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float4 t = *(const float4*)(bi + 8 * k);
      v[4 * k] = sum[b][4 * k] + t.x; v[4 * k + 1] = sum[b][4 * k + 1] + t.y; v[4 * k + 2] = sum[b][4 * k + 2] + t.z; v[4 * k + 3] = sum[b][4 * k + 3] + t.w;
    }
    if (c.res3) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if constexpr (BF16) {
          v[4 * k] += __uint_as_float(old[k].x << 16); v[4 * k + 1] += __uint_as_float(old[k].x & 0xffff0000u);
          v[4 * k + 2] += __uint_as_float(old[k].y << 16); v[4 * k + 3] += __uint_as_float(old[k].y & 0xffff0000u);
        } else {
          v[4 * k] += __uint_as_float(old[k].x); v[4 * k + 1] += __uint_as_float(old[k].y); v[4 * k + 2] += __uint_as_float(old[k].z); v[4 * k + 3] += __uint_as_float(old[k].w);
        }
      }
    }
    apply_act(v, c.act3);
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = inside ? v[k] : 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if constexpr (BF16) *(uint2*)(at + 8 * k * ES) = make_uint2(pack_bf16_rne(v[4 * k], v[4 * k + 1]), pack_bf16_rne(v[4 * k + 2], v[4 * k + 3]));
      else *(float4*)(at + 8 * k * ES) = make_float4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
    }
  }
  __syncthreads();

  const auto yrsrc = __builtin_amdgcn_make_buffer_rsrc(c.y3, 0, p.M * (kChainWide * ES), 0x00027000);
  auto store_wide = [&]() {
    uint4 out[NV];
#pragma unroll
    for (int r = 0; r < NV; ++r) {
      const int v = tid + r * NT;
      out[r] = *(const uint4*)(wide + v / ROW_VECS * WIDE + v % ROW_VECS * 16);
    }
#pragma unroll
    for (int r = 0; r < NV; ++r) put_at(yrsrc, at0 + (tid + r * NT) * 16, out[r]);
  };
  if (c.n1 == 0) {
    store_wide();
    return;
  }
  f32x16 acc[2] = {f32x16(0.f), f32x16(0.f)};
#pragma unroll
  for (int u = 0; u < U1; ++u) {
    const Split8 a = pixels_of(wide + li * WIDE, u0 + u);
#pragma unroll
    for (int k = 0; k < (BF16 ? 1 : 6); ++k)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[j] = mfma_bf16(a.p[PA[k]], w1[u][j][PB[k]], acc[j]);
  }
  store_wide();
  if constexpr (!BF16) {
    if (__builtin_expect(out_of_range(acc), 0)) {  // (the epilogue's second walk would find `wide` gone)
      ConvArgs x = ConvArgs();  // one row of 32 pixels in LDS
      x.x = wide; x.w = c.w1; x.H = 1; x.W = x.M = 32; x.Cin = WIDE / 4; x.kh = x.kw = x.stride = 1; x.S = 2 * S1;
      x.mg_wo = x.mg_cin = 1;  // (every pixel and every k is below Wo and Cin)
      const bool small = all_small(acc);
      const f32x16 had[2] = {acc[0], acc[1]};
      plain_products<3, 32, 1, 2>(x, DwFusedArgs(), 0, 0, 2 * u0, 2 * U1, acc);
#pragma unroll
      for (int j = 0; j < 2; ++j) take_second(small, had[j], acc[j]);
    }
  }
  __syncthreads();  // the partial tiles come where `wide` was
  fin.template finish<fin.kNoWalk>(q, DwFusedArgs(), acc, lds, m0, 0, 0, 0, 0);
}

// ---- pointwise layers: one thread per (output pixel, 16-byte channel vector) ----------------------------------------------
//
// Bound by the trip to memory, not by bytes: a layer of MobileNetV2 has one to two waves per SIMD and nothing to hide a load
// behind.  With the filter size known at compile time every load of a window is in flight at once (one trip instead of one per
// tap), and the thread's place comes from multiplications.  fp32 on 128 CUs: depthwise 14x14x384 3.29 -> 2.16 us, 28x28x192
// 3.48 -> 2.88, 7x7x960 3.33 -> 2.16; 3x3 pooling of 112x112x64 3.55 -> 2.34, 2x2 pooling of 224x224x64 3.80 -> 2.77
// (an empty launch: 1.5).  K = 0: any other filter size, and tensors whose byte
// offsets do not fit 31 bits, tap by tap.
// Workgroups L, L + 8, L + 16, ... run on one XCD: it gets a band of consecutive rows, so that the rows a band's windows
// share come from memory into its L2 once.
struct Point {
  int c0, m, oy, ox;  // first channel, output pixel
  bool ok;
};
template <bool BF16, typename Args>
__device__ __forceinline__ Point point_of(const Args& a, const PointPlace& at, const int L, const int tid) {
  const uint32_t idx = ((uint32_t)(L & 7) * at.per_xcd + (uint32_t)(L >> 3)) * 256u + (uint32_t)tid;
  const uint32_t cvn = (uint32_t)a.C / (BF16 ? 8 : 4);
  const uint32_t m = at.mg_cv == kNoMagic ? idx / cvn : (uint32_t)fast_div((int)idx, at.mg_cv);
  Point t;
  t.m = (int)m;
  t.c0 = (int)(idx - m * cvn) * (BF16 ? 8 : 4);
  t.ok = m < (uint32_t)a.Ho * (uint32_t)a.Wo;
  t.oy = at.mg_wo == kNoMagic ? (int)(m / (uint32_t)a.Wo) : fast_div((int)m, at.mg_wo);
  t.ox = t.m - t.oy * a.Wo;
  return t;
}
template <bool BF16, typename Args>
__device__ __forceinline__ Point point_of(const Args& a, const uint32_t idx) {  // any filter size: threads in order
  const uint32_t cvn = (uint32_t)a.C / (BF16 ? 8 : 4), m = idx / cvn;
  Point t;
  t.m = (int)m;
  t.c0 = (int)(idx - m * cvn) * (BF16 ? 8 : 4);
  t.ok = m < (uint32_t)a.Ho * (uint32_t)a.Wo;
  t.oy = (int)(m / (uint32_t)a.Wo);
  t.ox = t.m - t.oy * a.Wo;
  return t;
}

// depthwise convolution
template <bool BF16, int K>
__device__ __forceinline__ void dwconv_point(const DwArgs& a, const Point& t) {
  constexpr int VEC = BF16 ? 8 : 4;
  constexpr int ES = BF16 ? 2 : 4;
  if (!t.ok) return;
  float acc[VEC];
  const unsigned char* xb = (const unsigned char*)a.x;
  const unsigned char* wb = (const unsigned char*)a.w;
  const int iy0 = t.oy * a.stride - a.pad, ix0 = t.ox * a.stride - a.pad;
  if constexpr (K > 0) {
    const int step = a.C * ES, first = (iy0 * a.W + ix0) * step + t.c0 * ES;  // byte offsets (may start outside the image)
    uint4 xv[K * K], wv[K * K];
    bool in[K * K];
#pragma unroll
    for (int i = 0; i < K * K; ++i) {
      const int iy = iy0 + i / K, ix = ix0 + i % K;
      in[i] = (unsigned)iy < (unsigned)a.H && (unsigned)ix < (unsigned)a.W;
      xv[i] = *(const uint4*)(xb + (uint32_t)(in[i] ? first + (i / K * a.W + i % K) * step : 0));  // always a valid address
      wv[i] = *(const uint4*)(wb + (uint32_t)(t.c0 * ES + i * step));
    }
#pragma unroll
    for (int q = 0; q < VEC / 4; ++q) {
      const float4 b = *(const float4*)(a.bias + t.c0 + 4 * q);
      acc[4 * q] = b.x; acc[4 * q + 1] = b.y; acc[4 * q + 2] = b.z; acc[4 * q + 3] = b.w;
    }
#pragma unroll
    for (int j = 0; j < K * K; ++j) {
      float xf[VEC], wf[VEC];
      unpack<BF16>(xv[j], xf);
      unpack<BF16>(wv[j], wf);
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[i] = in[j] ? fmaf(xf[i], wf[i], acc[i]) : acc[i];
    }
  } else {
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] = a.bias[t.c0 + i];
    for (int ky = 0; ky < a.k; ++ky) {
      const int iy = iy0 + ky;
      if ((unsigned)iy >= (unsigned)a.H) continue;
      for (int kx = 0; kx < a.k; ++kx) {
        const int ix = ix0 + kx;
        if ((unsigned)ix >= (unsigned)a.W) continue;
        float xf[VEC], wf[VEC];
        unpack<BF16>(*(const uint4*)(xb + ((size_t)(iy * a.W + ix) * a.C + t.c0) * ES), xf);
        unpack<BF16>(*(const uint4*)(wb + ((size_t)(ky * a.k + kx) * a.C + t.c0) * ES), wf);
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[i] = fmaf(xf[i], wf[i], acc[i]);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < VEC; ++i) acc[i] = apply_act(acc[i], a.act);
  put((unsigned char*)a.y + ((size_t)t.m * a.C + t.c0) * ES, pack<BF16>(acc));
}

// max pooling: padding acts as -inf
template <bool BF16, int K>
__device__ __forceinline__ void maxpool_point(const PoolArgs& a, const Point& t) {
  constexpr int VEC = BF16 ? 8 : 4;
  constexpr int ES = BF16 ? 2 : 4;
  if (!t.ok) return;
  float best[VEC];
#pragma unroll
  for (int i = 0; i < VEC; ++i) best[i] = -INFINITY;
  const unsigned char* xb = (const unsigned char*)a.x;
  const int iy0 = t.oy * a.stride - a.pad, ix0 = t.ox * a.stride - a.pad;
  if constexpr (K > 0) {
    const int step = a.C * ES, first = (iy0 * a.W + ix0) * step + t.c0 * ES;  // byte offsets (may start outside the image)
    uint4 xv[K * K];
    bool in[K * K];
#pragma unroll
    for (int i = 0; i < K * K; ++i) {
      const int iy = iy0 + i / K, ix = ix0 + i % K;
      in[i] = (unsigned)iy < (unsigned)a.H && (unsigned)ix < (unsigned)a.W;
      xv[i] = *(const uint4*)(xb + (uint32_t)(in[i] ? first + (i / K * a.W + i % K) * step : 0));  // always a valid address
    }
#pragma unroll
    for (int j = 0; j < K * K; ++j) {
      float xf[VEC];
      unpack<BF16>(xv[j], xf);
#pragma unroll
      for (int i = 0; i < VEC; ++i) best[i] = in[j] ? fmaxf(best[i], xf[i]) : best[i];
    }
  } else {
    for (int ky = 0; ky < a.k; ++ky) {
      const int iy = iy0 + ky;
      if ((unsigned)iy >= (unsigned)a.H) continue;
      for (int kx = 0; kx < a.k; ++kx) {
        const int ix = ix0 + kx;
        if ((unsigned)ix >= (unsigned)a.W) continue;
        float xf[VEC];
        unpack<BF16>(*(const uint4*)(xb + ((size_t)(iy * a.W + ix) * a.C + t.c0) * ES), xf);
#pragma unroll
        for (int i = 0; i < VEC; ++i) best[i] = fmaxf(best[i], xf[i]);
      }
    }
  }
  put((unsigned char*)a.y + ((size_t)t.m * a.C + t.c0) * ES, pack<BF16>(best));
}

// ---- global average pooling: 64 channels per 256 threads, 4 threads per channel over the pixels, LDS sum ------------
// tid: the thread's number among the 256 of channel group `group`; part: their LDS.  Every thread of the workgroup calls it.
template <bool BF16>
__device__ __forceinline__ void gavgpool_group(const PoolArgs& a, const int group, const int tid, float (*part)[64]) {
  const int cl = tid & 63, q = tid >> 6;
  const int c = group * 64 + cl;
  const int hw = a.H * a.W;
  float s = 0.f;
  if (c < a.C) {
    int i = q;
    for (; i + 24 < hw; i += 28) {  // seven loads in flight (a 7 x 7 map: two trips to memory)
      float v[7];
#pragma unroll
      for (int u = 0; u < 7; ++u) v[u] = load_elem<BF16>(a.x, (size_t)(i + 4 * u) * a.C + c);
#pragma unroll
      for (int u = 0; u < 7; ++u) s += v[u];
    }
    float v[6];
#pragma unroll
    for (int u = 0; u < 6; ++u) v[u] = load_elem<BF16>(a.x, (size_t)min(i + 4 * u, hw - 1) * a.C + c);
#pragma unroll
    for (int u = 0; u < 6; ++u) s += i + 4 * u < hw ? v[u] : 0.f;
  }
  part[q][cl] = s;
  __syncthreads();
  if (q == 0 && c < a.C) put_elem<BF16>(a.y, c, (part[0][cl] + part[1][cl] + part[2][cl] + part[3][cl]) / (float)a.k);
}

// ---- FC, batch 1: one wave per output, 16-byte loads along K, butterfly reduction ------------------------------------
template <bool BF16>
__device__ __forceinline__ void fc_row(const FcArgs& a, const int n, const int lane) {
  constexpr int VEC = BF16 ? 8 : 4;
  constexpr int ES = BF16 ? 2 : 4;
  if (n >= a.Ns) return;
  if (n >= a.N) {  // pad element of the output vector
    if (lane == 0) put_elem<BF16>(a.y, n, 0.f);
    return;
  }
  const unsigned char* wrow = (const unsigned char*)a.w + (size_t)n * a.K * ES;
  const unsigned char* xb = (const unsigned char*)a.x;
  const int nvec = a.K / VEC;
  float bias = a.bias[n];  // (behind the sums it would be one more trip to memory)
  // Short rows are latency-bound: four independent 16-byte weight loads in flight per lane, each with its own partial sum.
  // Long rows (VGG-16's first FC: 100 KB per wave, 411 MB in all) are pure streaming and run at the memory system's
  // rate with one load per lane (bf16, rows half as long: two); more loads in flight slowed them down (measured: 84 -> 110 us).
  // A matrix that the last cache cannot hold from one frame to the next is read past it (stream), so that it does not drive
  // out the other layers' weights and tensors: VGG-16 on 128 CUs, fp32 570 -> 531 us a frame, bf16 316 -> 292 with one load
  // per lane, 286 with two (fp32 with two: 552; a row per workgroup instead of per wave: 557 and 284).
  float acc4[4] = {0.f, 0.f, 0.f, 0.f};
  int v = lane;
  if (nvec <= 2048) {
    for (; v + 192 < nvec; v += 256) {
      uint4 wq[4], xq[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) wq[u] = *(const uint4*)(wrow + (size_t)(v + 64 * u) * 16);
#pragma unroll
      for (int u = 0; u < 4; ++u) xq[u] = *(const uint4*)(xb + (size_t)(v + 64 * u) * 16);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        float wv[VEC], xv[VEC];
        unpack<BF16>(wq[u], wv);
        unpack<BF16>(xq[u], xv);
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc4[u] = fmaf(wv[i], xv[i], acc4[u]);
      }
    }
  }
  if (a.stream) {
    constexpr int U = BF16 ? 2 : 1;
    for (; v + 64 * (U - 1) < nvec; v += 64 * U) {
      uint4 wq[U], xq[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        wq[u] = __builtin_bit_cast(uint4, __builtin_nontemporal_load((const u32x4 __attribute__((address_space(1)))*)(uintptr_t)(wrow + (size_t)(v + 64 * u) * 16)));
#pragma unroll
      for (int u = 0; u < U; ++u) xq[u] = *(const uint4*)(xb + (size_t)(v + 64 * u) * 16);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float wv[VEC], xv[VEC];
        unpack<BF16>(wq[u], wv);
        unpack<BF16>(xq[u], xv);
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc4[u] = fmaf(wv[i], xv[i], acc4[u]);
      }
    }
  }
  for (; v < nvec; v += 64) {
    float wv[VEC], xv[VEC];
    unpack<BF16>(*(const uint4*)(wrow + (size_t)v * 16), wv);
    unpack<BF16>(*(const uint4*)(xb + (size_t)v * 16), xv);
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc4[0] = fmaf(wv[i], xv[i], acc4[0]);
  }
  float acc = (acc4[0] + acc4[1]) + (acc4[2] + acc4[3]);
  asm volatile("" : "+v"(bias));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if (lane == 0) {
    const float v = apply_act(acc + bias, a.act);
    if (a.out_f32) put((float*)a.y + n, v);
    else put_elem<BF16>(a.y, n, v);
  }
}

}  // namespace daris

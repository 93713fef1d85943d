// Device-side helpers that the kernels of every code object share: element conversions and vector packing, index division,
// and the products of fp32 operands on the bf16 matrix instructions.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace daris {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// ---- element helpers ------------------------------------------------------------------------------------------

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

// float -> bfloat16 bits, round to nearest, ties to even; NaN stays a quiet NaN.  One v_cvt_pk_bf16_f32.
__device__ __forceinline__ uint32_t pack_bf16_rne(float a, float b) {
  f32x2 v;
  v.x = a;
  v.y = b;
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) { return pack_bf16_rne(f, 0.f) & 0xffffu; }

__device__ __forceinline__ float apply_act(float v, int act) {
  if (act == 1) v = fmaxf(v, 0.f);
  else if (act == 2) v = fminf(fmaxf(v, 0.f), 6.f);
  return v;
}

// The same for many values, with one branch and one instruction each (v_med3_f32: NaN becomes 0, as with fmaxf).
template <int N>
__device__ __forceinline__ void apply_act(float (&v)[N], int act) {
  if (act == 0) return;
  const float most = act == 2 ? 6.f : INFINITY;
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = __builtin_amdgcn_fmed3f(v[i], 0.f, most);
}

template <bool BF16>
__device__ __forceinline__ float load_elem(const void* p, size_t i) {
  if (BF16) return bf16_bits_to_f32(((const uint16_t*)p)[i]);
  return ((const float*)p)[i];
}

// What a kernel leaves for the next one is written through to where all eight XCDs see it, and every wave waits for its
// stores before it ends.  The packets of a stage therefore need no release fence (a write-back of eight L2s after every
// kernel: 0.5 us of the 5 us that a launch of a small layer takes).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void put(void* p, const uint4& v) {
  __builtin_amdgcn_global_store_b128((u32x4 __attribute__((address_space(1)))*)p, __builtin_bit_cast(u32x4, v), "agent");
}
__device__ __forceinline__ void put(void* p, const float4& v) { put(p, __builtin_bit_cast(uint4, v)); }
__device__ __forceinline__ void put(void* p, const uint2& v) {
  __hip_atomic_store((uint64_t __attribute__((address_space(1)))*)p, __builtin_bit_cast(uint64_t, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <bool BF16>
__device__ __forceinline__ void put_elem(void* p, size_t i, float v) {
  if (BF16) __hip_atomic_store((uint16_t*)p + i, (uint16_t)f32_to_bf16_bits(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else put((float*)p + i, v);
}
// ... at byte offset `at` of a tensor behind a buffer descriptor (past its end: dropped)
constexpr int kWriteThrough = 16;  // sc1
__device__ __forceinline__ void put_at(__amdgpu_buffer_rsrc_t t, int at, const uint4& v) { __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), t, at, 0, kWriteThrough); }
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void put_at(__amdgpu_buffer_rsrc_t t, int at, const uint2& v) { __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), t, at, 0, kWriteThrough); }
__device__ __forceinline__ void puts_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// n / d for 0 <= n with n * d < 2^32, through the host-made multiplier magic = floor(2^32 / d) + 1 (0 stands for d = 1):
// the quotient is the high word of n * magic, a handful of cycles instead of the ~40-instruction division sequence.
__device__ __forceinline__ int fast_div(int n, uint32_t magic) { return magic ? (int)__umulhi((uint32_t)n, magic) : n; }

// A kernel's arguments (or any constant block) in one batch of scalar loads.  Left to itself the compiler fetches the
// fields it needs first, branches, and fetches the rest: one more trip to memory, 0.25 us per launch.
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef i32x8 i32x8_a4 __attribute__((aligned(4)));
typedef i32x4 i32x4_a4 __attribute__((aligned(4)));
typedef i32x2 i32x2_a4 __attribute__((aligned(4)));
typedef const unsigned char __attribute__((address_space(4))) * ConstPtr;

template <typename T>
__device__ __forceinline__ T grab(ConstPtr src) {
  constexpr int N = sizeof(T), W = N / 32, R = N % 32;  // vectors of eight words, then one of four, then one of two
  static_assert(N % 8 == 0 && W >= 1 && W <= 5 && R % 8 == 0 && R != 8, "no such argument block");
  struct {
    i32x8 w[W];
    i32x4 q;
    i32x2 d;
  } v;
#pragma unroll
  for (int i = 0; i < W; ++i) v.w[i] = *(const i32x8_a4 __attribute__((address_space(4)))*)(src + 32 * i);
  if constexpr (R >= 16) v.q = *(const i32x4_a4 __attribute__((address_space(4)))*)(src + 32 * W);
  if constexpr (R == 24) v.d = *(const i32x2_a4 __attribute__((address_space(4)))*)(src + 32 * W + 16);
  if constexpr (W == 5) asm volatile("" : "+s"(v.w[0]), "+s"(v.w[1]), "+s"(v.w[2]), "+s"(v.w[3]), "+s"(v.w[4]));
  else if constexpr (W == 2 && R == 24) asm volatile("" : "+s"(v.w[0]), "+s"(v.w[1]), "+s"(v.q), "+s"(v.d));
  else if constexpr (W == 2 && R == 0) asm volatile("" : "+s"(v.w[0]), "+s"(v.w[1]));
  else if constexpr (W == 1 && R == 24) asm volatile("" : "+s"(v.w[0]), "+s"(v.q), "+s"(v.d));
  else if constexpr (W == 1 && R == 16) asm volatile("" : "+s"(v.w[0]), "+s"(v.q));
  else static_assert(N == 0, "no such argument block");
  T t;
  __builtin_memcpy(&t, &v, N);
  return t;
}

// A pointer known to be one to device memory: loads through a pointer of unknown kind would count as LDS accesses as well,
// and a wait for LDS would wait for them.  (The compiler knows it by itself only for a kernel's own parameters.)
template <typename T>
__device__ __forceinline__ T* in_memory(T* p) {
  return (T*)(T __attribute__((address_space(1)))*)(uintptr_t)p;
}

// v if ok, else all zero bits; component-wise so that it stays a register select (a select between two uint4
// objects would be done through their addresses and push the access to scratch / flat memory).
__device__ __forceinline__ uint4 keep_if(bool ok, uint4 v) {
  v.x = ok ? v.x : 0u;
  v.y = ok ? v.y : 0u;
  v.z = ok ? v.z : 0u;
  v.w = ok ? v.w : 0u;
  return v;
}

// Unpack one 16-byte vector into VEC floats (4 for fp32, 8 for bf16).
template <bool BF16>
__device__ __forceinline__ void unpack(const uint4& v, float* o) {
  if (BF16) {
    o[0] = __uint_as_float(v.x << 16); o[1] = __uint_as_float(v.x & 0xffff0000u);
    o[2] = __uint_as_float(v.y << 16); o[3] = __uint_as_float(v.y & 0xffff0000u);
    o[4] = __uint_as_float(v.z << 16); o[5] = __uint_as_float(v.z & 0xffff0000u);
    o[6] = __uint_as_float(v.w << 16); o[7] = __uint_as_float(v.w & 0xffff0000u);
  } else {
    o[0] = __uint_as_float(v.x); o[1] = __uint_as_float(v.y); o[2] = __uint_as_float(v.z); o[3] = __uint_as_float(v.w);
  }
}

template <bool BF16>
__device__ __forceinline__ uint4 pack(const float* o) {
  uint4 v;
  if (BF16) {
    v.x = pack_bf16_rne(o[0], o[1]);
    v.y = pack_bf16_rne(o[2], o[3]);
    v.z = pack_bf16_rne(o[4], o[5]);
    v.w = pack_bf16_rne(o[6], o[7]);
  } else {
    v.x = __float_as_uint(o[0]); v.y = __float_as_uint(o[1]); v.z = __float_as_uint(o[2]); v.w = __float_as_uint(o[3]);
  }
  return v;
}

// ---- fp32 products on the bf16 matrix instructions ---------------------------------------------------------------------
//
// An fp32 number has 24 significant bits, a bf16 number 8 and the same exponents: a finite fp32 number of 2^-110 and more is the
// exact sum of three bf16 numbers x1 + x2 + x3, each at most 2^-7 of the one before; below that the third part, and from 2^-118
// on the second, is rounded to the smallest bf16 number (2^-133), so that up to 2^-134 is lost.  A product of two such sums has
// nine terms, each exact in fp32; the six largest (x1y1, x1y2, x2y1, x1y3, x2y2, x3y1) leave out at most 2^-23 of |xy|, with no
// bias, where the fp32 instruction loses nothing before it adds (but measured on sums of 4608 terms against float64 its error is
// the larger one: 4.2e-7 against 3.6e-7).  v_mfma_f32_32x32x16_bf16 does in 32
// cycles what v_mfma_f32_32x32x2_f32 does in 512, so the six take 3/8 of the matrix time.  Accumulation is fp32 as before.
// The first part of an activation is cut off (a rounded one could overflow), all other parts are rounded to nearest even;
// the weights' parts are made at registration.  (An infinite operand gives
// NaN; plain_products in layer_bodies.h puts that right, and a tile of pixels so small that they lose bits.)
struct Split8 {
  uint4 p[3];  // eight consecutive k: first, second, third parts
};

// lo = elements 0..3, hi = elements 4..7
__device__ __forceinline__ Split8 split8(const uint4& lo, const uint4& hi) {
  const uint32_t in[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
  uint32_t out[3][4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t u0 = in[2 * i], u1 = in[2 * i + 1];
    out[0][i] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);  // the upper halves
    const float r0 = __uint_as_float(u0) - __uint_as_float(u0 & 0xffff0000u), r1 = __uint_as_float(u1) - __uint_as_float(u1 & 0xffff0000u);
    const uint32_t m = pack_bf16_rne(r0, r1);
    out[1][i] = m;
    out[2][i] = pack_bf16_rne(r0 - __uint_as_float(m << 16), r1 - __uint_as_float(m & 0xffff0000u));
  }
  Split8 s;
#pragma unroll
  for (int q = 0; q < 3; ++q) s.p[q] = make_uint4(out[q][0], out[q][1], out[q][2], out[q][3]);
  return s;
}

// The parts of four consecutive values.
struct Split4 {
  uint2 p[3];
};
__device__ __forceinline__ Split4 split4(const uint4& v) {
  const Split8 s = split8(v, make_uint4(0u, 0u, 0u, 0u));
  Split4 t;
#pragma unroll
  for (int q = 0; q < 3; ++q) t.p[q] = make_uint2(s.p[q].x, s.p[q].y);
  return t;
}

__device__ __forceinline__ f32x16 mfma_bf16(const uint4& a, const uint4& b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

}  // namespace daris

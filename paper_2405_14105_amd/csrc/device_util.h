// Device helpers: bf16 conversion, hi/lo split, MFMA wrappers, fragment
// loads and pack stores.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace dsi {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// two fp32 -> two bf16 bit patterns (a in the low half), round to nearest
// even: one v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t f2bf_pair(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}
__device__ __forceinline__ uint16_t f2bf_bits(float f) { return (uint16_t)f2bf_pair(f, 0.f); }
__device__ __forceinline__ float bf_bits2f(uint16_t b) {
  return __uint_as_float(((uint32_t)b) << 16);
}

// split x into bf16 hi + bf16 lo with x ~= hi + lo (to ~2^-17 relative)
__device__ __forceinline__ void split_bf16(float x, uint16_t& hi, uint16_t& lo) {
  hi = f2bf_bits(x);
  lo = f2bf_bits(x - bf_bits2f(hi));
}
// the same for a pair: hi and lo hold a's half low, b's half high
__device__ __forceinline__ void split_pair(float a, float b, uint32_t& hi, uint32_t& lo) {
  hi = f2bf_pair(a, b);
  lo = f2bf_pair(a - __uint_as_float(hi << 16), b - __uint_as_float(hi & 0xFFFF0000u));
}
// eight values as MFMA fragments
__device__ __forceinline__ void split8(const float (&v)[8], u32x4& hi, u32x4& lo) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    uint32_t h, l;
    split_pair(v[2 * e], v[2 * e + 1], h, l);
    hi[e] = h;
    lo[e] = l;
  }
}

__device__ __forceinline__ f32x4 mfma_bf16(const bf16x8& a, const bf16x8& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_f32(float a, float b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16x8 as_bf16x8(const u32x4& v) {
  return __builtin_bit_cast(bf16x8, v);
}

// the maximum / sum over the four lanes l, l ^ 16, l ^ 32, l ^ 48 (the lanes
// that hold one query's keys): two VALU lane swaps, where a shuffle goes
// through LDS.  The sum adds in the order of __shfl_xor 16, then 32.
__device__ __forceinline__ float max_over_16_32(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float sum_over_16_32(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// 8 fp32 values (two 16-byte loads)
struct F8 {
  float4 a, b;
};
__device__ __forceinline__ float f8_get(const F8& v, int e) {
  switch (e) {
    case 0: return v.a.x; case 1: return v.a.y; case 2: return v.a.z; case 3: return v.a.w;
    case 4: return v.b.x; case 5: return v.b.y; case 6: return v.b.z; default: return v.b.w;
  }
}

// store one activation value into a pack at (token m, feature f)
__device__ __forceinline__ size_t pack_index(int Kb, int m, int f) {
  const int mt = m >> 4, kb = f >> 5, grp = (f & 31) >> 3, e = f & 7;
  const int lane = (m & 15) + 16 * grp;
  return (((size_t)mt * Kb + kb) * 64 + lane) * 8 + e;
}
__device__ __forceinline__ void pack_store(const PackRef& p, int wtype, int m, int f, float v) {
  const size_t idx = pack_index(p.Kb, m, f);
  if (wtype == W_BF16) {
    uint16_t hi, lo;
    split_bf16(v, hi, lo);
    ((uint16_t*)p.hi)[idx] = hi;
    ((uint16_t*)p.lo)[idx] = lo;
  } else {
    ((float*)p.hi)[idx] = v;
  }
}

// store features f, f + 1 (f even) of token m
__device__ __forceinline__ void pack_store2(const PackRef& p, int wtype, int m, int f, float a, float b) {
  const size_t idx = pack_index(p.Kb, m, f);
  if (wtype == W_BF16) {
    uint32_t h, l;
    split_pair(a, b, h, l);
    *(uint32_t*)((uint16_t*)p.hi + idx) = h;
    *(uint32_t*)((uint16_t*)p.lo + idx) = l;
  } else {
    *(float2*)((float*)p.hi + idx) = float2{a, b};
  }
}

// store 4 consecutive features f0..f0+3 (f0 % 4 == 0) of token m: 8 bytes
// per half for bf16 packs, 16 bytes for fp32 packs
__device__ __forceinline__ void pack_store4(const PackRef& p, int wtype, int m, int f0, const float* v) {
  const size_t idx = pack_index(p.Kb, m, f0);
  if (wtype == W_BF16) {
    uint2 h, l;
    split_pair(v[0], v[1], h.x, l.x);
    split_pair(v[2], v[3], h.y, l.y);
    *(uint2*)((uint16_t*)p.hi + idx) = h;
    *(uint2*)((uint16_t*)p.lo + idx) = l;
  } else {
    *(float4*)((float*)p.hi + idx) = float4{v[0], v[1], v[2], v[3]};
  }
}

// store 8 consecutive features f0..f0+7 (f0 % 8 == 0) of token m: one
// 16-byte store per half for bf16 packs, two for fp32 packs
__device__ __forceinline__ void pack_store8(const PackRef& p, int wtype, int m, int f0, const float* v) {
  const size_t idx = pack_index(p.Kb, m, f0);
  if (wtype == W_BF16) {
    const float y[8] = {v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]};
    u32x4 h, l;
    split8(y, h, l);
    *(u32x4*)((uint16_t*)p.hi + idx) = h;
    *(u32x4*)((uint16_t*)p.lo + idx) = l;
  } else {
    float* d = (float*)p.hi + idx;
    *(float4*)d = float4{v[0], v[1], v[2], v[3]};
    *(float4*)(d + 4) = float4{v[4], v[5], v[6], v[7]};
  }
}

// cache policy of a buffer load: device scope (sc1)
constexpr int kSc1 = 16;

// Device-scope (sc1) 16-byte store: written through to the device's
// coherence point, for partial results that another workgroup of the same
// kernel reads with device-scope loads after an arrival counter says they
// are complete (the writer waits for vmcnt(0) before counting).  One wide
// store instead of four device-scope dword stores.
__device__ __forceinline__ void store4_device(float* p, f32x4 v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc1" ::"v"(p), "v"(v) : "memory");
}

__device__ __forceinline__ float silu_f(float x) { return x / (1.0f + __expf(-x)); }

}  // namespace dsi

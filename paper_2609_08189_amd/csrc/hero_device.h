// Device-side helpers shared by the HeRo kernels (gfx950 / CDNA4, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hero {

typedef uint16_t bf16_t;  // bfloat16 storage (bit pattern)

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;

__device__ __forceinline__ float bf16_to_f32(bf16_t b) {
  return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

// Round to nearest even (v_cvt_pk_bf16_f32 on gfx950).
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  return __builtin_bit_cast(bf16_t, static_cast<__bf16>(f));
}

template <typename T> struct io;
template <> struct io<float> {
  static __device__ __forceinline__ float ld(const float* p) { return *p; }
  static __device__ __forceinline__ void st(float* p, float v) { *p = v; }
};
template <> struct io<bf16_t> {
  static __device__ __forceinline__ float ld(const bf16_t* p) { return bf16_to_f32(*p); }
  static __device__ __forceinline__ void st(bf16_t* p, float v) { *p = f32_to_bf16(v); }
};

template <typename T>
__device__ __forceinline__ float ldf(const T* p) { return io<T>::ld(p); }
template <typename T>
__device__ __forceinline__ void stf(T* p, float v) { io<T>::st(p, v); }

// 8 consecutive elements as fp32 (16-byte aligned for bf16, 32-byte for fp32).
__device__ __forceinline__ void ld8(const bf16_t* p, float* o) {
  u32x4 v = *reinterpret_cast<const u32x4*>(p);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    o[2 * i] = __uint_as_float(v[i] << 16);
    o[2 * i + 1] = __uint_as_float(v[i] & 0xffff0000u);
  }
}
__device__ __forceinline__ void ld8(const float* p, float* o) {
  f32x4 a = *reinterpret_cast<const f32x4*>(p);
  f32x4 b = *reinterpret_cast<const f32x4*>(p + 4);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    o[i] = a[i];
    o[4 + i] = b[i];
  }
}
__device__ __forceinline__ void st8(bf16_t* p, const float* v) {
  u32x4 w;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    w[i] = static_cast<uint32_t>(f32_to_bf16(v[2 * i])) |
           (static_cast<uint32_t>(f32_to_bf16(v[2 * i + 1])) << 16);
  *reinterpret_cast<u32x4*>(p) = w;
}
__device__ __forceinline__ void st8(float* p, const float* v) {
  f32x4 a, b;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    a[i] = v[i];
    b[i] = v[4 + i];
  }
  *reinterpret_cast<f32x4*>(p) = a;
  *reinterpret_cast<f32x4*>(p + 4) = b;
}

// Eight consecutive elements as loaded (bf16 stays packed: 4 registers per chunk).
template <typename T> struct Raw8;
template <> struct Raw8<bf16_t> {
  u32x4 v;
  __device__ __forceinline__ void load(const bf16_t* p) { v = *reinterpret_cast<const u32x4*>(p); }
  __device__ __forceinline__ float operator[](int i) const {
    const uint32_t w = v[i >> 1];
    return __uint_as_float((i & 1) ? (w & 0xffff0000u) : (w << 16));
  }
};
template <> struct Raw8<float> {
  f32x4 a, b;
  __device__ __forceinline__ void load(const float* p) {
    a = *reinterpret_cast<const f32x4*>(p);
    b = *reinterpret_cast<const f32x4*>(p + 4);
  }
  __device__ __forceinline__ float operator[](int i) const { return i < 4 ? a[i] : b[i - 4]; }
};

// order-preserving image of an fp32 value (-0 and +0 map to the same key)
__device__ __forceinline__ uint32_t order_key(float f) {
  uint32_t b = __float_as_uint(f);
  if (b == 0x80000000u) b = 0u;
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

__device__ __forceinline__ float sigmoidf_(float x) { return 1.0f / (1.0f + expf(-x)); }
__device__ __forceinline__ float siluf_(float x) { return x / (1.0f + expf(-x)); }
// ELU(x) + 1, with exp(x) evaluated directly below zero.
__device__ __forceinline__ float phif_(float x) { return x > 0.0f ? x + 1.0f : expf(x); }

// Sum over the aligned group of PI lanes a lane is in (a power of two up to 32), left in every lane
// of the group: DPP moves up to 16 lanes (quad swaps, then mirrors of rows whose quads agree).
template <int PI>
__device__ __forceinline__ float group_sum(float v) {
  static_assert(PI >= 1 && PI <= 32 && (PI & (PI - 1)) == 0, "lanes");
#define HERO_DPP_ADD(ctrl) v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), ctrl, 0xf, 0xf, true))
  if constexpr (PI >= 2) HERO_DPP_ADD(0xB1);    // lanes 1 0 3 2 of each quad
  if constexpr (PI >= 4) HERO_DPP_ADD(0x4E);    // lanes 2 3 0 1
  if constexpr (PI >= 8) HERO_DPP_ADD(0x141);   // half rows mirrored
  if constexpr (PI >= 16) HERO_DPP_ADD(0x140);  // rows mirrored
#undef HERO_DPP_ADD
  if constexpr (PI >= 32) v += __shfl_xor(v, 16, kWave);
  return v;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

}  // namespace hero

// Cache rows in registers: 16-byte pieces of bf16 or float32 elements.
#pragma once
#include "fg_common.h"

template <int ESIZE>
__device__ __forceinline__ void fg_unpack(const u32x4& v, float* f);
template <>
__device__ __forceinline__ void fg_unpack<2>(const u32x4& v, float* f) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[2 * i] = fg_bf16_lo(v[i]);
    f[2 * i + 1] = fg_bf16_hi(v[i]);
  }
}
template <>
__device__ __forceinline__ void fg_unpack<4>(const u32x4& v, float* f) {
#pragma unroll
  for (int i = 0; i < 4; ++i) f[i] = __uint_as_float(v[i]);
}

// Dot product of the 8 bf16 pairs of two 16-byte chunks with float accumulation: four
// two-element dot instructions instead of eight unpacks and eight multiply-adds. Serves the
// output path only (the cumulative scores use the float64 logits).
__device__ __forceinline__ float fg_dot_bf16x8(const u32x4& a, const u32x4& b) {
  float acc = 0.f;
  // (pairs taken from the 8-element vectors by shuffles: handed bit-cast dwords of the 128-bit
  // vectors, the compiler of ROCm 7.2 selects element 0 for all four instructions)
  const bf16x8 av = __builtin_bit_cast(bf16x8, a), bv = __builtin_bit_cast(bf16x8, b);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(av, av, 0, 1), __builtin_shufflevector(bv, bv, 0, 1), acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(av, av, 2, 3), __builtin_shufflevector(bv, bv, 2, 3), acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(av, av, 4, 5), __builtin_shufflevector(bv, bv, 4, 5), acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(av, av, 6, 7), __builtin_shufflevector(bv, bv, 6, 7), acc, false);
  return acc;
}

template <int ESIZE>
__device__ __forceinline__ void fg_store_out(void* out, size_t idx, float v);
template <>
__device__ __forceinline__ void fg_store_out<2>(void* out, size_t idx, float v) {
  static_cast<uint16_t*>(out)[idx] = (uint16_t)fg_f32_to_bf16_bits(v);
}
template <>
__device__ __forceinline__ void fg_store_out<4>(void* out, size_t idx, float v) {
  static_cast<float*>(out)[idx] = v;
}
